"""Timed cases of the pruning library: what a program that prunes visual tokens has it do.

Every case is one call (or the two calls that belong together) through
paper_2608_25332_amd.provip with outputs and workspace allocated once, as a
serving loop keeps them.  The sizes are those of the library's own workloads
(LLaVA-1.5-7B: 576 tokens of width 4096, 32 heads x 128; LLaVA-NeXT AnyRes: 5
tiles of 576; a 13B backbone with 8 frames; the tiny fp32 set) and generic
ragged ones.

  step         pv_prune_pipeline, the whole pruning step; with "graph" it is
               captured once and replayed, as a decoder at batch 1 runs it
  dedup        pv_prune_dedup alone (pruning before the LLM, with the merge)
  text         pv_critical_text, the selection of the critical text tokens
  heads        pv_visual_heads and, on its list, pv_prune_head_aware (a
               shallow pruning layer)
  score        pv_prune_head_aware on a given head list
  gather       pv_prune_gather_batch, the compaction of hidden rows, K and V
  progressive  pv_prune_progressive, the three-stage schedule
"""

from __future__ import annotations

import math

import torch

from paper_2608_25332_amd import provip

DEV = "cuda:0"
DT = {"bf16": torch.bfloat16, "f32": torch.float32}
ESZ = {"bf16": 2, "f32": 4}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: the tiny fp32 set, straight from Python, where
        # only the call itself and its launches count
        dict(name="step-tiny-f32", op="step", scene="plain", dtype="f32", B=1, Nv=64, Nt=16, d=256,
             H=4, hd=64, n_heads=1, N1=32, N2=16, graph=False),
        # one LLaVA-1.5-7B request at the latency that matters for decoding:
        # the step inside a captured graph
        dict(name="step-7b-b1", op="step", scene="image", dtype="bf16", B=1, Nv=576, Nt=64, d=4096,
             H=32, hd=128, n_heads=4, N1=192, N2=64, graph=True),
        # a batch of such requests
        dict(name="step-7b-b16", op="step", scene="image", dtype="bf16", B=16, Nv=576, Nt=64,
             d=4096, H=32, hd=128, n_heads=4, N1=192, N2=64, graph=False),
        # the largest step: eight frames through a 13B-width backbone
        dict(name="step-13b-video", op="step", scene="video", dtype="bf16", B=2, Nv=4608, Nt=128,
             d=5120, H=40, hd=128, n_heads=5, N1=1152, N2=512, graph=False),
        # AnyRes tiles, pruning before the LLM on its own (the layers up to
        # the pruning layer run between it and the rest of the step)
        dict(name="dedup-hires", op="dedup", scene="tiles", dtype="bf16", B=4, Nv=2880, Nt=128,
             d=4096, N1=960, masked=False),
        # fp32 embeddings of an odd width and token count, critical rows only
        dict(name="dedup-f32-ragged", op="dedup", scene="image", dtype="f32", B=3, Nv=1037, Nt=37,
             d=1000, N1=345, masked=True),
        # critical text tokens of a batch of long prompts
        dict(name="text-b16", op="text", dtype="bf16", B=16, Nt=300, d=4096),
        # shallow pruning layer at the AnyRes size: which heads are visual,
        # then the score on them
        dict(name="heads-hires", op="heads", dtype="bf16", B=4, H=32, Nt=128, N=960, hd=128,
             n_heads=6, N2=320, masked=True),
        # middle pruning layer of a large batch: every head
        dict(name="score-all-heads", op="score", dtype="bf16", B=64, H=32, Nt=64, N=192, hd=128,
             n_heads=32, N2=64, lse=False),
        # a backbone with 80-wide heads, odd prompt and token counts, on the
        # model's own softmax domain
        dict(name="score-hd80-lse", op="score", dtype="bf16", B=8, H=32, Nt=37, N=577, hd=80,
             n_heads=6, N2=193, lse=True),
        # hidden rows, K and V of the kept tokens of a batch
        dict(name="gather-b16", op="gather", dtype="bf16", B=16, N=576, d=4096, H=32, hd=128,
             k=192),
        # the whole schedule for a small batch of requests
        dict(name="progressive-7b-b8", op="progressive", scene="image", dtype="bf16", B=8, Nv=576,
             Nt=64, d=4096, H=32, hd=128, N1=192, n_vis=6, N2=64, N3=32),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: the ranges between the listed ones, odd sizes among them."""
    op = rng.choice(["step", "step", "dedup", "dedup", "text", "heads", "score", "score", "gather",
                     "progressive"])
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    # widths in earnest are multiples of 64; one in four is only a multiple of 8
    d = _log(rng, 32, 640) * 8 if rng.random() < 0.25 else _log(rng, 4, 80) * 64
    hd = rng.choice([64, 64, 80, 96, 128, 128, 128, 128])
    H = rng.choice([4, 8, 16, 28, 32, 40])
    Nt = _log(rng, 8, 160)
    Nv = _log(rng, 64, 4608)
    cap = 2 if dtype == "bf16" else 1
    # the batch: at most about 40 M elements of visual rows (fp32: 8 M)
    most = max(1, min(48, (40 if cap == 2 else 8) * 1000000 // (Nv * d)))
    B = _log(rng, 1, most)
    N1 = max(2, int(Nv * rng.uniform(0.2, 0.5)))
    if dtype == "f32":  # the matrix cores multiply fp32 at a sixteenth of the bf16 rate
        while 2.0 * B * (Nv - N1) * N1 * d > 4e9 and Nv > 64:
            Nv, N1 = max(64, Nv * 2 // 3), max(2, N1 * 2 // 3)
    else:
        while 2.0 * B * (Nv - N1) * N1 * d > 7.5e10 and Nv > 64:
            Nv, N1 = max(64, Nv * 2 // 3), max(2, N1 * 2 // 3)
    scene = "plain" if Nv < 128 else rng.choice(["image", "tiles", "video"])
    N2 = max(1, int(N1 * rng.uniform(0.2, 0.6)))
    while 2.0 * B * H * Nv * hd * ESZ[dtype] > 180e6 and B > 1:
        B = max(1, B // 2)
    if op == "step":
        return dict(op=op, scene=scene, dtype=dtype, B=B, Nv=Nv, Nt=Nt, d=d, H=H, hd=hd,
                    n_heads=rng.randint(1, max(1, H // 4)), N1=N1, N2=N2, graph=B <= 2)
    if op == "dedup":
        return dict(op=op, scene=scene, dtype=dtype, B=B, Nv=Nv, Nt=Nt, d=d, N1=N1,
                    masked=rng.random() < 0.5)
    if op == "text":
        return dict(op=op, dtype=dtype, B=_log(rng, 1, 16), Nt=_log(rng, 8, 300), d=d)
    if op == "gather":
        return dict(op=op, dtype=dtype, B=B, N=Nv, d=d, H=H, hd=hd, k=N1)
    if op == "progressive":
        return dict(op=op, scene=scene, dtype=dtype, B=min(B, 8), Nv=Nv, Nt=Nt, d=d, H=H, hd=hd,
                    N1=N1, n_vis=rng.randint(1, max(1, H // 4)), N2=N2, N3=max(1, N2 // 2))
    N = _log(rng, 32, 1152)
    Bq = _log(rng, 1, max(1, min(64, 1600000 // (H * N))))
    if dtype == "f32":
        Bq = max(1, Bq // 2)
    N2 = max(1, N // 3)
    if op == "heads":
        return dict(op=op, dtype=dtype, B=min(Bq, 8), H=H, Nt=Nt, N=N, hd=hd,
                    n_heads=rng.randint(1, max(1, H // 4)), N2=N2, masked=rng.random() < 0.5)
    return dict(op=op, dtype=dtype, B=Bq, H=H, Nt=Nt, N=N, hd=hd,
                n_heads=H if rng.random() < 0.5 else rng.randint(1, max(1, H // 4)), N2=N2,
                lse=rng.random() < 0.5)


# ---------------------------------------------------------------------------
# inputs, drawn on the GPU from the seed alone (elementwise arithmetic only,
# so that every process gets the same bits)
# ---------------------------------------------------------------------------
class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device=DEV)

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, device=DEV)

    def order(self, rows, n):
        return torch.argsort(self.uniform(rows, n), dim=1)


def _fields(dr, B, n, rank=8):
    """[rank, B, n]: smooth fields over the smallest square grid that holds n
    tokens, sums of three 2-D cosines of at most two cycles."""
    side = max(1, math.isqrt(n - 1) + 1)
    at = torch.arange(n, device=DEV)
    y, x = (at // side).float(), (at % side).float()
    out = torch.zeros(rank, B, n, device=DEV)
    for _ in range(3):
        k = torch.floor(dr.uniform(2, rank, B, 1) * 3)
        ph = dr.uniform(rank, B, 1)
        out += torch.cos(2 * math.pi * ((k[0] * y + (k[1] + (k[0] + k[1] == 0)) * x) / side + ph))
    return out


def _smooth(dr, B, n, d, rank=8, weight=0.6):
    """[B, n, d]: N(0, 1) noise plus a rank-8 smooth field (neighbouring tokens
    have a cosine of about 0.8)."""
    f = _fields(dr, B, n, rank)
    v = dr.normal(B, n, d)
    for r in range(rank):
        v.addcmul_(f[r].unsqueeze(2), dr.normal(B, 1, d), value=weight)
    return v


def _visual(dr, scene, B, Nv, d, dtype):
    """Connector outputs: plain N(0, 1) rows with a few exact duplicates, one
    image, five image tiles with near-duplicate tokens in each, or eight
    frames that differ from the first by noise."""
    if scene == "plain":
        v = dr.normal(B, Nv, d)
        n = Nv // 8
        v[:, Nv - n:] = v[:, :n]
    elif scene == "image":
        v = _smooth(dr, B, Nv, d)
    elif scene == "tiles":
        per = (Nv + 4) // 5
        v = torch.cat([_smooth(dr, B, per, d) for _ in range(5)], 1)[:, :Nv].contiguous()
        n = Nv // 10  # followers of the token before them
        at = dr.order(1, max(1, Nv // 2 - 1))[0, :n] * 2 + 1
        v[:, at] = v[:, at - 1] + 0.2 * dr.normal(B, at.numel(), d)
    else:
        per = (Nv + 7) // 8
        first = _smooth(dr, B, per, d)
        v = torch.cat([first] + [first + 0.4 * dr.normal(B, per, d) for _ in range(7)], 1)
        v = v[:, :Nv].contiguous()
    return v.to(DT[dtype])


def _text(dr, B, Nt, d, dtype):
    """Prompt embeddings: a few shared topics, repeated tokens, norms around 2."""
    topic = dr.normal(B, 6, d)
    pick = torch.floor(dr.uniform(B, Nt) * 6).long()
    e = dr.normal(B, Nt, d) + 0.8 * torch.gather(topic, 1, pick.unsqueeze(2).expand(B, Nt, d))
    n = Nt // 6
    if n:
        e[:, Nt - n:] = e[:, :n]  # words that occur twice
    scale = (0.5 + dr.uniform(B, Nt, 1)) * (1.6 / math.sqrt(d))
    return (e * scale).to(DT[dtype])


def _queries(dr, B, H, Nt, hd, dtype):
    """Text-query rows; some heads attend sharply, others nearly evenly."""
    return (dr.normal(B, H, Nt, hd) * (0.4 + 1.8 * dr.uniform(B, H, 1, 1))).to(DT[dtype])


def _keys(dr, B, H, N, hd, dtype):
    return dr.normal(B, H, N, hd).to(DT[dtype])


def _head_list(dr, B, H, n):
    return torch.sort(dr.order(B, H)[:, :n], dim=1)[0].to(torch.int32)


def _mask(dr, B, Nt):
    return (dr.uniform(B, Nt) < 0.6).to(torch.int32)


def prepare(case, seed):
    c, dr = dict(case), _Draw(seed)
    op, dtype, B = c["op"], c["dtype"], c["B"]
    s = {"c": c}
    if op == "step":
        s["vis"] = _visual(dr, c["scene"], B, c["Nv"], c["d"], dtype)
        s["anchors"] = _text(dr, B, c["Nt"], c["d"], dtype)
        s["q"] = _queries(dr, B, c["H"], c["Nt"], c["hd"], dtype)
        s["k"] = _keys(dr, B, c["H"], c["Nv"], c["hd"], dtype)
        s["v"] = _keys(dr, B, c["H"], c["Nv"], c["hd"], dtype)
        s["heads"] = _head_list(dr, B, c["H"], c["n_heads"]).cpu().numpy()
        # the first call allocates the outputs and the workspace the program keeps
        o = _step(s, None, None)
        s["ws"] = o.pop("workspace")
        s["out"] = o
        if c["graph"]:
            torch.cuda.synchronize()
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                _step(s, s["out"], s["ws"])
    elif op == "dedup":
        s["vis"] = _visual(dr, c["scene"], B, c["Nv"], c["d"], dtype)
        s["anchors"] = _text(dr, B, c["Nt"], c["d"], dtype)
        s["mask"] = _mask(dr, B, c["Nt"]) if c["masked"] else None
        o = provip.pv_prune_dedup(s["vis"], s["anchors"], c["N1"], anchor_mask=s["mask"])
        s["ws"] = o["workspace"]
        s["out"] = {k: o[k] for k in ("kept", "score", "assign", "merged")}
    elif op == "text":
        s["text"] = _text(dr, B, c["Nt"], c["d"], dtype)
        o = provip.pv_critical_text(s["text"])
        s["ws"] = o["workspace"]
        s["out"] = {k: o[k] for k in ("mask", "count", "r")}
    elif op == "heads":
        s["q"] = _queries(dr, B, c["H"], c["Nt"], c["hd"], dtype)
        s["k"] = _keys(dr, B, c["H"], c["N"], c["hd"], dtype)
        s["mask"] = _mask(dr, B, c["Nt"]) if c["masked"] else None
        o = provip.pv_visual_heads(s["q"], s["k"], c["n_heads"], row_mask=s["mask"])
        s["ws"] = o["workspace"]
        s["out"] = {k: o[k] for k in ("heads", "conf")}
        o = provip.pv_prune_head_aware(s["q"], s["k"], s["out"]["heads"], c["N2"])
        s["ws2"] = o["workspace"]
        s["out2"] = {k: o[k] for k in ("kept", "score")}
    elif op == "score":
        s["q"] = _queries(dr, B, c["H"], c["Nt"], c["hd"], dtype)
        s["k"] = _keys(dr, B, c["H"], c["N"], c["hd"], dtype)
        s["heads"] = _head_list(dr, B, c["H"], c["n_heads"]).cpu().numpy()
        # as much weight on the system and text keys as the visual keys have, give or take
        s["lse"] = (math.log(c["N"]) + dr.normal(B, c["H"], c["Nt"])) if c["lse"] else None
        o = provip.pv_prune_head_aware(s["q"], s["k"], s["heads"], c["N2"], row_lse=s["lse"])
        s["ws"] = o["workspace"]
        s["out"] = {k: o[k] for k in ("kept", "score")}
    elif op == "gather":
        s["srcs"] = [dr.normal(B, c["N"], c["d"]).to(DT[dtype]),
                     _keys(dr, B, c["H"], c["N"], c["hd"], dtype),
                     _keys(dr, B, c["H"], c["N"], c["hd"], dtype)]
        s["idx"] = torch.sort(dr.order(B, c["N"])[:, :c["k"]], dim=1)[0].to(torch.int32)
        s["outs"] = provip.pv_prune_gather_batch(s["srcs"], s["idx"])
    else:
        s["text"] = _text(dr, B, c["Nt"], c["d"], dtype)
        s["vis"] = _visual(dr, c["scene"], B, c["Nv"], c["d"], dtype)
        for n in ("s", "m"):
            s["q_" + n] = _queries(dr, B, c["H"], c["Nt"], c["hd"], dtype)
            s["k_" + n] = _keys(dr, B, c["H"], c["Nv"], c["hd"], dtype)
        o = _progressive(s, None, None)
        s["ws"] = o.pop("workspace")
        s["out"] = o
    return s


def _step(s, out, ws):
    c = s["c"]
    return provip.pv_prune_pipeline(s["vis"], s["anchors"], s["q"], s["k"], s["v"], s["heads"],
                                    c["N1"], c["N2"], out=out, workspace=ws)


def _progressive(s, out, ws):
    c = s["c"]
    return provip.pv_prune_progressive(s["text"], s["vis"], s["q_s"], s["k_s"], s["q_m"], s["k_m"],
                                       c["N1"], c["n_vis"], c["N2"], c["N3"], out=out, workspace=ws)


def run(s):
    c = s["c"]
    op = c["op"]
    if op == "step":
        if c["graph"]:
            s["graph"].replay()
        else:
            _step(s, s["out"], s["ws"])
        return s["out"]
    if op == "dedup":
        provip.pv_prune_dedup(s["vis"], s["anchors"], c["N1"], out=s["out"], workspace=s["ws"],
                              anchor_mask=s["mask"])
        return s["out"]
    if op == "text":
        provip.pv_critical_text(s["text"], out=s["out"], workspace=s["ws"])
        return s["out"]
    if op == "heads":
        provip.pv_visual_heads(s["q"], s["k"], c["n_heads"], out=s["out"], workspace=s["ws"],
                               row_mask=s["mask"])
        provip.pv_prune_head_aware(s["q"], s["k"], s["out"]["heads"], c["N2"], out=s["out2"],
                                   workspace=s["ws2"])
        return {"layer": s["out"], "pruned": s["out2"]}
    if op == "score":
        provip.pv_prune_head_aware(s["q"], s["k"], s["heads"], c["N2"], out=s["out"],
                                   workspace=s["ws"], row_lse=s["lse"])
        return s["out"]
    if op == "gather":
        provip.pv_prune_gather_batch(s["srcs"], s["idx"], outs=s["outs"])
        return s["outs"]
    _progressive(s, s["out"], s["ws"])
    return s["out"]


# ---------------------------------------------------------------------------
# the work a pass cannot do without: each input read once where the method
# needs it (the kept rows of K and V, the selected heads), each output written
# once
# ---------------------------------------------------------------------------
def _dedup_work(B, Nv, Nt, d, N1, e):
    return (B * ((Nv + Nt) * d * e + N1 * d * e + 4 * (N1 + 2 * Nv)),
            2.0 * B * d * (Nt * Nv + (Nv - N1) * N1))


def _score_work(B, n_heads, Nt, N, hd, N2, e):
    return B * (n_heads * (Nt + N) * hd * e + 4 * (N + N2)), 2.0 * B * n_heads * Nt * N * hd


def work(case):
    c = case
    B, e = c["B"], ESZ[c["dtype"]]
    op = c["op"]
    if op == "text":
        by, fl = B * (c["Nt"] * c["d"] * e + 8 * c["Nt"] + 4), 2.0 * B * c["Nt"] ** 2 * c["d"]
    elif op == "gather":
        by, fl = 2 * B * c["k"] * (c["d"] + 2 * c["H"] * c["hd"]) * e + 4 * B * c["k"], 0.0
    elif op == "score":
        by, fl = _score_work(B, c["n_heads"], c["Nt"], c["N"], c["hd"], c["N2"], e)
        by += 4 * B * c["n_heads"] * c["Nt"] if c["lse"] else 0
    elif op == "heads":
        by, fl = _score_work(B, c["H"], c["Nt"], c["N"], c["hd"], c["N2"], e)
        by += 4 * B * (c["H"] + c["n_heads"])
        fl += 2.0 * B * c["n_heads"] * c["Nt"] * c["N"] * c["hd"]
    else:
        by, fl = _dedup_work(B, c["Nv"], c["Nt"], c["d"], c["N1"], e)
        if op == "step":
            N1, N2 = c["N1"], c["N2"]
            fl += 2.0 * B * c["n_heads"] * c["Nt"] * N1 * c["hd"]
            # queries of the selected heads; K and V of the N1 kept in and
            # out; the N2 kept rows of the hidden states, K and V out
            by += B * e * (c["n_heads"] * c["Nt"] * c["hd"] + 4 * c["H"] * N1 * c["hd"]
                           + N2 * (c["d"] + 2 * c["H"] * c["hd"])) + 4 * B * (N1 + N2)
        elif op == "progressive":
            N1, N2, N3 = c["N1"], c["N2"], c["N3"]
            fl += 2.0 * B * c["Nt"] * (c["Nt"] * c["d"] + c["hd"] * (
                c["H"] * N1 + c["n_vis"] * N1 + c["H"] * N2))
            by += B * e * (c["H"] * c["hd"] * (2 * c["Nt"] + N1 + N2) + (N2 + N3) * c["d"])
            by += 4 * B * (c["Nt"] + c["n_vis"] + c["H"] + N1 + 2 * N2 + N3)
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    """fp32 scores: against 64 bits the sums are off by 1e-7 to 2e-7 (2-norm),
    so two orders of summation differ by up to twice that.  Rows written in
    bf16: off by 1.3e-3 from the rounding alone, and a sum in another order may
    round one value to its neighbour (2^-7 of it).  Scores closer than that may
    change a kept index."""
    op = case["op"]
    if op == "gather":
        return "exact"
    if op in ("text", "heads", "score") or case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 2e-5, "differ": 0.005}
    return {"rel": 5e-3, "max": 0.03, "differ": 0.002}


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _topk64(score, k):
    """Indices of the k largest, lower index first among equals (to 1e-12), ascending."""
    at = torch.sort(torch.round(score * 1e12), dim=-1, descending=True, stable=True)[1]
    return torch.sort(at[..., :k])[0]


def _unit64(x):
    x = x.double()
    n = x.norm(dim=-1, keepdim=True)
    return torch.where(n > 0, x / n, torch.zeros_like(x))


def _dedup64(vis, anchors, N1, mask):
    kept, score, assign, merged = [], [], [], []
    for b in range(vis.shape[0]):
        v, a = _unit64(vis[b]), _unit64(anchors[b])
        if mask is not None and bool(mask[b].any()):
            a = a[mask[b].bool()]
        m = torch.mm(a, v.t())
        p = (m - m.mean(1, keepdim=True)).max(0)[0]
        kp = _topk64(p, N1)
        g = torch.mm(v, v[kp].t())
        slots = torch.arange(N1, device=vis.device)
        # the lowest slot of equal maxima; a kept token takes its own
        asg = torch.where(g >= g.max(1, keepdim=True)[0] - 1e-12, slots, N1).min(1)[0]
        asg[kp] = slots
        tot = torch.zeros(N1, vis.shape[2], dtype=torch.float64, device=vis.device)
        tot.index_add_(0, asg, vis[b].double())
        cnt = torch.bincount(asg, minlength=N1).double()
        kept.append(kp.int())
        score.append(p)
        assign.append(asg.int())
        merged.append(tot / cnt.unsqueeze(1))
    return [torch.stack(t) for t in (kept, score, assign, merged)]


def _map64(q, k, lse):
    """Softmax rows [Nt, N] of one head, the other keys' log-sum-exp in the normaliser."""
    s = torch.mm(q.double(), k.double().t()) / math.sqrt(q.shape[-1])
    if lse is not None:
        return torch.softmax(torch.cat([s, lse.double().unsqueeze(1)], 1), 1)[:, :-1]
    return torch.softmax(s, 1)


def _score64(q, k, heads, N2, lse=None):
    v = []
    for b in range(q.shape[0]):
        v.append(sum(_map64(q[b, h], k[b, h], None if lse is None else lse[b, h]).mean(0)
                     for h in [int(x) for x in heads[b]]) / len(heads[b]))
    v = torch.stack(v)
    return _topk64(v, N2).int(), v


def _rows64(src, idx):
    """The rows idx [B, k] of [B, N, d] or, in every head, of [B, H, N, hd]."""
    return torch.stack([src[b].index_select(src.dim() - 3, idx[b].long())
                        for b in range(src.shape[0])])


def _text64(text):
    mask, count, r = [], [], []
    for e in text:
        e = e.double()
        x = torch.softmax(torch.mm(e, e.t()), 1).mean(0)
        m = x > x.mean()
        if not bool(m.any()):
            m = torch.ones_like(m)
        mask.append(m.int())
        count.append(m.sum().int())
        r.append(x)
    return torch.stack(mask), torch.stack(count), torch.stack(r)


def _conf64(q, k, n_vis, mask):
    conf = []
    for b in range(q.shape[0]):
        use = mask[b].bool() if mask is not None and bool(mask[b].any()) else slice(None)
        conf.append(torch.stack([_map64(q[b, h], k[b, h], None)[use].var(1, unbiased=False).sum()
                                 for h in range(q.shape[1])]))
    conf = torch.stack(conf)
    return _topk64(conf, n_vis).int(), conf


def exact(case, seed):
    s = prepare(case, seed)
    c, op = s["c"], case["op"]
    if op == "gather":
        return [_rows64(t, s["idx"]).double() for t in s["srcs"]]
    if op == "text":
        m, n, r = _text64(s["text"])
        return {"mask": m, "count": n, "r": r}
    if op == "score":
        kept, v = _score64(s["q"], s["k"], s["heads"], c["N2"], s["lse"])
        return {"kept": kept, "score": v}
    if op == "heads":
        heads, conf = _conf64(s["q"], s["k"], c["n_heads"], s["mask"])
        kept, v = _score64(s["q"], s["k"], heads.cpu().numpy(), c["N2"])
        return {"layer": {"heads": heads, "conf": conf}, "pruned": {"kept": kept, "score": v}}
    if op == "dedup":
        kept, p, asg, merged = _dedup64(s["vis"], s["anchors"], c["N1"], s["mask"])
        return {"kept": kept, "score": p, "assign": asg, "merged": merged}
    if op == "step":
        kept, p, asg, merged = _dedup64(s["vis"], s["anchors"], c["N1"], None)
        k1, v1 = _rows64(s["k"], kept), _rows64(s["v"], kept)
        kept2, v = _score64(s["q"], k1, s["heads"], c["N2"])
        return {"kept1": kept, "score1": p, "assign": asg, "merged": merged, "k1": k1.double(),
                "v1": v1.double(), "kept2": kept2, "score2": v, "hidden2": _rows64(merged, kept2),
                "k2": _rows64(k1, kept2).double(), "v2": _rows64(v1, kept2).double()}
    mask, _, _ = _text64(s["text"])
    kept, _, asg, merged = _dedup64(s["vis"], s["text"], c["N1"], mask)
    ks = _rows64(s["k_s"], kept)
    heads, conf = _conf64(s["q_s"], ks, c["n_vis"], mask)
    l2, v2 = _score64(s["q_s"], ks, heads.cpu().numpy(), c["N2"])
    kept2 = torch.gather(kept, 1, l2.long())
    hidden2 = _rows64(merged, l2)
    every = [list(range(c["H"]))] * c["B"]
    l3, v3 = _score64(s["q_m"], _rows64(s["k_m"], kept2), every, c["N3"])
    return {"text_mask": mask, "kept1": kept, "assign": asg, "merged": merged, "vis_heads": heads,
            "conf": conf, "kept2": kept2, "score2": v2, "hidden2": hidden2,
            "kept3": torch.gather(kept2, 1, l3.long()), "score3": v3, "hidden3": _rows64(hidden2, l3)}
