"""The GEMM for grids of few output tiles (plans with 32-row tiles) against the oracle, at the
edges of its tiles, of its waves' K ranges and of its plan's rules.  Every product is exact in
float32, so Y differs from the float64 result by the rounding of at most K sums of partial
sums: normwise well below the repository's bound of 1e-5 for float32 outputs."""
import numpy as np
import pytest

from oracle import formats as F
from oracle import resq as Q
from synth import activations, bf16_bits_to_f32, rng_tree, weights
from _gpu_util import assert_close, dev_bf16, host, log

FMTS = ["mxfp4", "hif4"]
# m, d, n: one row, row 31 / 32 / 33; one column tile, a ragged last one; fewer K steps than
# waves, one more, many; an MXFP4 half step (d % 64 == 32)
CASES = [(1, 64, 1), (31, 512, 33), (32, 576, 64), (33, 1088, 95), (100, 2048, 2080), (255, 512, 1000),
         (256, 2048, 2048), (8, 2048, 16416), (64, 640, 16400), (128, 256, 4608), (3, 32800, 40)]


def _plan(P, fmt, m, d, n):
    return P.gemm_plan(fmt, m, n, d, True)


def test_cases_cover_every_streamed_plan():
    """CPU: the cases reach every tile width, wave count and K split that the plans use."""
    import paper_2607_26515_amd as P
    seen = set()
    for fmt in FMTS:
        for m, d, n in CASES:
            p = _plan(P, fmt, m, d // 64 * 64, n)
            if p["tile"].startswith("32x"):
                seen.add((fmt, p["tile"], p["kgroups"], p["ksplit"] > 1))
    assert seen == {("mxfp4", "32x32", 8, False), ("mxfp4", "32x32", 8, True), ("mxfp4", "32x64", 8, False),
                    ("mxfp4", "32x64", 4, False), ("hif4", "32x32", 8, False), ("hif4", "32x32", 8, True),
                    ("hif4", "32x64", 8, False), ("hif4", "32x96", 8, False), ("hif4", "32x64", 4, False)}


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("sp", ["none", "2:4"])
@pytest.mark.parametrize("m,d,n", CASES)
def test_streamed_forward(fmt, sp, m, d, n):
    import torch
    import paper_2607_26515_amd as P
    d = d if fmt == "mxfp4" else d // 64 * 64
    log(f"streamed gemm {fmt} {sp} m={m} d={d} n={n} plan={_plan(P, fmt, m, d, n)}")
    rx, rw = rng_tree(m + d + n, 2)
    xb, wb = activations(rx, m, d, 0.01, 50.0), weights(rw, n, d)
    qc, qs = P.quantize(dev_bf16(wb), fmt)
    wp = P.prepare_weights(qc, qs, fmt)
    x = dev_bf16(xb)
    y = torch.full((m, n + 3), 7.0, dtype=torch.float32, device="cuda")  # row stride n + 3
    P.linear_fwd_prepared(x, wp, n, fmt, sp, y=y[:, :n])
    yb = P.linear_fwd_prepared(x, wp, n, fmt, sp, out="bf16")
    o = Q.resq_quantize_residual(fmt, sp, bf16_bits_to_f32(xb))
    cols = np.unique(np.r_[0:min(n, 300), max(0, n - 300):n])  # the oracle's columns
    w = F.dequantize(fmt, *F.quantize(fmt, bf16_bits_to_f32(wb[cols])))
    want = (o["xhat"] + o.get("srhat", 0.0)) @ w.T
    got = host(y)
    assert_close(got[:, :n][:, cols], want, f"Y {fmt} {sp}")
    assert (got[:, n:] == 7.0).all(), "a store left its row"
    assert np.array_equal(host(yb).view(np.uint16), Q.round_to_bf16(got[:, :n]))


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("m,d,n", CASES)
def test_streamed_every_column_tile_and_same_bits(fmt, m, d, n):
    """Every 29th column, so that each 32-column tile is compared, with the columns' places in a
    workgroup's 32, 64 or 96 all occurring; and a second call into another Y gives the same bits."""
    import torch
    import paper_2607_26515_amd as P
    d = d if fmt == "mxfp4" else d // 64 * 64
    log(f"streamed gemm columns {fmt} m={m} d={d} n={n} plan={_plan(P, fmt, m, d, n)}")
    rx, rw = rng_tree(3 * m + d + n, 2)
    xb, wb = activations(rx, m, d, 0.01, 50.0), weights(rw, n, d)
    qc, qs = P.quantize(dev_bf16(wb), fmt)
    wp = P.prepare_weights(qc, qs, fmt)
    x = dev_bf16(xb)
    y = P.linear_fwd_prepared(x, wp, n, fmt, "2:4", y=torch.full((m, n), float("nan"), device="cuda"))
    y2 = P.linear_fwd_prepared(x, wp, n, fmt, "2:4", y=torch.full((m, n), 7.0, device="cuda"))
    assert torch.equal(y.view(torch.int32), y2.view(torch.int32)), "two identical calls differ"
    cols = np.arange((m + d) % 29 % n, n, 29)
    o = Q.resq_quantize_residual(fmt, "2:4", bf16_bits_to_f32(xb))
    w = F.dequantize(fmt, *F.quantize(fmt, bf16_bits_to_f32(wb[cols])))
    assert_close(host(y)[:, cols], (o["xhat"] + o["srhat"]) @ w.T, f"Y {fmt}")
