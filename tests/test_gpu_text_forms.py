"""The forms of the critical-text call against the oracle: the streaming and
the split-k self-similarity (tiles of the upper triangle, ragged edges), and
the one- and three-launch ranking on both sides of every row size."""

from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_2608_25332_amd import workloads as W
from parity_util import TAU, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("B,Nt,d,dt", [
    (16, 257, 2056, "bf16"),   # streaming: 5 x 5 tiles, the last one row and column wide
    (40, 100, 1000, "bf16"),   # streaming: 2 x 2 tiles
    (200, 33, 4096, "bf16"),   # streaming: one tile per sample
    (1, 64, 512, "bf16"), (2, 65, 512, "bf16"), (1, 128, 264, "bf16"), (1, 129, 512, "f32"),
    (2, 256, 256, "bf16"), (1, 511, 256, "f32"), (1, 513, 256, "bf16")])
def test_text_forms(B, Nt, d, dt):
    from paper_2608_25332_amd import provip
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[text] B={B} Nt={Nt} d={d} {dt}", flush=True)
    rng = np.random.default_rng(Nt + d)
    text = (rng.standard_normal((B, Nt, d)) * (1.7 / np.sqrt(d))).astype(np.float32)
    if dt == "bf16":
        text = W.bf16_round(text)
    r = provip.pv_critical_text(to_dev(text, dt))
    torch.cuda.synchronize()
    mask, count, rg = to_host(r["mask"]), to_host(r["count"]), to_host(r["r"])
    some = sorted({0, B // 2, B - 1})
    ref, mask_ref, _ = oracle.critical_text(text[some])
    # logits to about 30 with an fp32 error of 1e-7 of them: 3e-6 of an exponential
    assert rel_err(rg[some], ref) <= 1e-5
    assert np.array_equal(count, mask.sum(1))
    for q, b in enumerate(some):
        sure = np.abs(ref[q] - ref[q].mean()) > TAU[dt] * ref[q].max()
        assert np.array_equal(mask[b][sure], mask_ref[q][sure])
    again = provip.pv_critical_text(to_dev(text, dt), want_r=False)
    torch.cuda.synchronize()
    assert np.array_equal(to_host(again["mask"]), mask)
