"""The forms of the head-confidence kernel against the oracle: rows per
workgroup 16, 32 and 64, one and two wave sets over the keys, ragged rows and
keys, and logits that outgrow the running reference between chunks."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_25332_amd import workloads as W
from parity_util import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (B, H, Nt, N, hd, dtype): 64 rows per workgroup with one wave set (N <= 256) and two,
# 32 rows, 16 rows (few heads; or wide fp32 rows beside which no more query rows fit)
CONF = [(4, 16, 65, 256, 64, "bf16"), (4, 16, 65, 257, 64, "bf16"), (2, 64, 33, 700, 80, "bf16"),
        (8, 16, 17, 130, 128, "bf16"), (4, 32, 32, 65, 128, "f32"), (1, 8, 64, 321, 128, "bf16"),
        (2, 64, 40, 100, 256, "f32"), (1, 128, 64, 1, 32, "bf16"), (4, 32, 48, 63, 96, "bf16")]


@pytest.mark.parametrize("B,H,Nt,N,hd,dt", CONF)
@pytest.mark.parametrize("grow", [False, True])
def test_head_conf_forms(B, H, Nt, N, hd, dt, grow):
    from paper_2608_25332_amd import provip
    print(f"[head_conf] B={B} H={H} Nt={Nt} N={N} hd={hd} {dt} grow={grow}", flush=True)
    rng = np.random.default_rng(Nt * 1000 + N + hd)
    q = rng.standard_normal((B, H, Nt, hd), dtype=np.float32)
    k = rng.standard_normal((B, H, N, hd), dtype=np.float32)
    if grow:  # later chunks hold logits tens of powers of two larger
        k *= (1.0 + 3.0 * (np.arange(N) // 64)[None, None, :, None]).astype(np.float32)
    if dt == "bf16":
        q, k = W.bf16_round(q), W.bf16_round(k)
    mask = (rng.random((B, Nt)) < 0.7).astype(np.int32)
    n_vis = max(1, H // 4)
    qd, kd = to_dev(q, dt), to_dev(k, dt)
    r = provip.pv_visual_heads(qd, kd, n_vis)
    m = provip.pv_visual_heads(qd, kd, n_vis, row_mask=torch.from_numpy(mask).to(qd.device))
    torch.cuda.synchronize()
    for b in {0, B - 1}:
        _, conf = oracle.visual_heads(q[b:b + 1], k[b:b + 1], n_vis)
        # logits of up to about 2^7 (2^10 grown) with an fp32 error of 2^-22 of
        # them: 2^-13 of an exponential at most, 1e-6 seen
        assert rel_err(to_host(r["conf"])[b], conf[0]) <= (2e-4 if grow else 1e-5)
        rows = mask[b].astype(bool) if mask[b].any() else slice(None)
        _, conf = oracle.visual_heads(q[b:b + 1][:, :, rows], k[b:b + 1], n_vis)
        assert rel_err(to_host(m["conf"])[b], conf[0]) <= (2e-4 if grow else 1e-5)
    for o in (r, m):  # the list is the top of the confidences written, ascending
        conf = to_host(o["conf"])
        order = np.argsort(-conf, axis=1, kind="stable")[:, :n_vis]
        assert np.array_equal(to_host(o["heads"]), np.sort(order, axis=1))


# (B, H, Nt, N, hd, n_heads, dtype): head widths between the streamed ones, in every form of
# the score: 16-row blocks with the logits held and with two passes, split keys, whole heads
WIDTHS = [(2, 4, 21, 65, 8, 2, "bf16"), (2, 4, 21, 300, 136, 2, "bf16"), (1, 2, 40, 2100, 104, 2, "bf16"),
          (1, 2, 18, 700, 248, 1, "f32"), (2, 4, 37, 321, 48, 3, "bf16"), (1, 4, 65, 257, 56, 3, "f32"),
          (32, 8, 63, 255, 120, 4, "bf16"), (64, 4, 17, 66, 40, 2, "bf16"), (64, 4, 33, 129, 24, 2, "f32")]


@pytest.mark.parametrize("B,H,Nt,N,hd,n_heads,dt", WIDTHS)
def test_head_widths_read_in_place(B, H, Nt, N, hd, n_heads, dt):
    """Q and K stand inside NaN: a piece read past the last row would spoil the sums, and one
    read past any other row would add the next row's elements."""
    from paper_2608_25332_amd import provip
    print(f"[head width] B={B} H={H} Nt={Nt} N={N} hd={hd} {dt}", flush=True)
    rng = np.random.default_rng(hd * 100 + N)
    q = rng.standard_normal((B, H, Nt, hd), dtype=np.float32)
    k = rng.standard_normal((B, H, N, hd), dtype=np.float32)
    if dt == "bf16":
        q, k = W.bf16_round(q), W.bf16_round(k)

    def inside_nan(x):
        d = to_dev(x, dt)
        buf = torch.full((d.numel() + 1024,), float("nan"), dtype=d.dtype, device=d.device)
        buf[512:512 + d.numel()] = d.reshape(-1)
        return buf[512:512 + d.numel()].view(d.shape)

    qd, kd = inside_nan(q), inside_nan(k)
    heads = np.stack([rng.permutation(H)[:n_heads] for _ in range(B)]).astype(np.int32)
    r = provip.pv_prune_head_aware(qd, kd, heads, max(1, N // 3))
    c = provip.pv_visual_heads(qd, kd, 1)
    torch.cuda.synchronize()
    for b in {0, B - 1}:
        _, v = oracle.head_aware(q[b:b + 1], k[b:b + 1], heads[b:b + 1], max(1, N // 3))
        assert rel_err(to_host(r["score"])[b], v[0]) <= 1e-5
        _, conf = oracle.visual_heads(q[b:b + 1], k[b:b + 1], 1)
        assert rel_err(to_host(c["conf"])[b], conf[0]) <= 1e-5
