"""resq_quantize along rows, bit for bit against the oracle, where its kernel can go wrong: float32
inputs on and one place around every rounding midpoint of every HiF4 grid (level-1 fraction,
level-2/3 shift, both signs) and at the saturation and zero ends; and the row kernel's edges
(rows around its step, one block per row, widths around its lane counts, unaligned rows and
outputs)."""
import numpy as np
import pytest

from oracle import formats as F
from _gpu_util import assert_codes_equal, assert_scales_equal, dev_bf16, dev_f32, log
from synth import activations, rng_tree

pytestmark = pytest.mark.gpu


def _check(P, x, t, fmt, what):
    qc, qs = P.quantize(t, fmt)
    oc, os_ = F.quantize(fmt, x)
    assert_codes_equal(qc, oc, what)
    assert_scales_equal(fmt, qs, os_, what)


def test_hif4_float32_midpoints():
    import paper_2607_26515_amd as P
    log("hif4 float32 midpoints")
    rows = []
    for e in (0, 1, 31, 45, 62):
        for m in range(4):
            s1 = np.float32(2.0 ** (e - 31) * (1 + m / 4))
            for b in range(3):
                step = np.float64(s1) / 4 * 2.0 ** -b
                mid = np.array([(j + 0.5) * step for j in range(8)], np.float32)  # exact
                vals = np.concatenate([mid, np.nextafter(mid, np.float32(0)), np.nextafter(mid, np.float32(1e38)),
                                       np.array([0.0, 7 * step], np.float32)])
                vals = vals[vals <= np.float32(7 * step)]  # the group keeps shift b
                row = np.zeros(64 * ((len(vals) + 2) // 3), np.float32)
                for i in range(0, len(vals), 3):
                    blk = row[64 * (i // 3):64 * (i // 3) + 64]
                    blk[0] = np.float32(1.75) * s1           # the block's maximum fixes level 1
                    blk[8:8 + len(vals[i:i + 3])] = vals[i:i + 3]
                    blk[11] = np.float32(7 * step)           # fixes the shift of this level-3 group
                    blk[12] = np.float32(7 * step) if b < 2 else np.float32(0)
                for sign in (1, -1):
                    rows.append(sign * row)
    width = max(len(r) for r in rows)
    x = np.stack([np.concatenate([r, np.zeros(width - len(r), np.float32)]) for r in rows])
    _check(P, x, dev_f32(x), "hif4", "midpoints")


@pytest.mark.parametrize("fmt", ["mxfp4", "hif4"])
@pytest.mark.parametrize("rows,cols", [(1, 64), (3, 448), (17, 512), (33, 576), (15, 2048), (5, 2112), (4097, 64)])
def test_row_kernel_edges(fmt, rows, cols):
    import torch
    import paper_2607_26515_amd as P
    from synth import bf16_bits_to_f32
    log(f"quant rows {fmt} {rows}x{cols}")
    for pad in (0, 4, 3):  # row strides that allow 16-byte, 8-byte and single loads
        xb = activations(rng_tree(rows + cols + pad, 1)[0], rows, cols + pad, 0.01, 50.0)
        x = bf16_bits_to_f32(xb)[:, :cols]
        _check(P, x, dev_bf16(xb)[:, :cols], fmt, f"bf16 pad {pad}")
        _check(P, x, dev_f32(bf16_bits_to_f32(xb))[:, :cols], fmt, f"f32 pad {pad}")
    # codes at an address that is only 2-byte aligned
    xb = activations(rng_tree(7, 1)[0], rows, cols, 0.01, 50.0)
    t = dev_bf16(xb)
    want, _ = P.quantize(t, fmt)
    buf = torch.zeros(rows * cols // 2 + 2, dtype=torch.uint8, device="cuda")
    sc = torch.zeros(rows * cols, dtype=torch.uint8, device="cuda")
    assert P.resq_quantize(P.FORMATS[fmt], t.data_ptr(), P.IN_BF16, rows, cols, cols, 1, buf.data_ptr() + 2,
                           sc.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    assert torch.equal(buf[2:].reshape(rows, cols // 2), want)


LANES = [(32, 32), (64, 32), (96, 16), (128, 16), (192, 8), (256, 8), (320, 4), (1024, 2), (1088, 1)]


@pytest.mark.parametrize("fmt,cols,step", [(f, c, s) for f in ("mxfp4", "hif4") for c, s in LANES if f == "mxfp4" or c % 64 == 0])
def test_row_kernel_lane_counts(fmt, cols, step):
    """Every number of lanes along a row (8 .. 256, widths that fill them and that do not) with row
    counts around the rows of a workgroup (`step`), one workgroup and several."""
    import paper_2607_26515_amd as P
    from synth import bf16_bits_to_f32
    for rows in sorted({1, step - 1, step, step + 1, 5 * step + 1} - {0}):
        log(f"quant rows lanes {fmt} {rows}x{cols}")
        xb = activations(rng_tree(1000 * rows + cols, 1)[0], rows, cols, 0.01, 50.0)
        _check(P, bf16_bits_to_f32(xb), dev_bf16(xb), fmt, f"{rows}x{cols}")
