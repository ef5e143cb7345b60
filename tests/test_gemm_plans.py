"""The GEMM's plans, as the host-side query reports them (CPU)."""
import itertools
import os
import subprocess
import sys

import pytest

import paper_2607_26515_amd as P

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("m,n", [(257, 25505), (331, 24150), (512, 12800), (896, 10240), (1555, 4640), (1664, 4224),
                                 (3853, 2636), (4080, 1559)])
@pytest.mark.parametrize("split", [False, True])
def test_hif4_eight_wave_tiles_only_within_the_cus(m, n, split):
    """A CU holds one workgroup of eight waves of the 128 x 192 HiF4 tile (its waves take more than
    128 registers) but two of four waves: more tiles than the 256 CUs run as four waves, all of
    them at once up to 512, instead of in two rounds."""
    tiles = -(-m // 128) * -(-n // 192)
    assert tiles > 256
    assert P.gemm_plan("hif4", m, n, 2048, split)["tile"] == "128x192"


def test_hif4_eight_wave_tiles_are_still_used():
    """Up to one workgroup per CU."""
    for m, n in itertools.product((256, 512, 1024), (4096, 12288, 24384)):
        tiles = -(-m // 128) * -(-n // 192)
        if 240 <= -(-m // 128) * -(-n // 128) and tiles <= 256:
            assert P.gemm_plan("hif4", m, n, 2048)["tile"] == "128x192_8w", (m, n)


def test_empty_products_have_plans_and_workspaces():
    """No rows or no columns, over every range of K that the plans tell apart: the queries answer (in
    a child process, since a division by the number of tiles would end this one)."""
    code = """
import paper_2607_26515_amd as P
for fmt in ("mxfp4", "hif4"):
    for m, n in ((0, 64), (64, 0), (0, 0), (0, 40000), (8192, 0)):
        for k in (0, 64, 8192, 32768, 1 << 20):
            for split in (False, True):
                assert P.gemm_plan(fmt, m, n, k, split)["ksplit"] == 1
            for op in range(7):
                P.resq_workspace_size(op, P.FORMATS[fmt], 2, m, k, n)
print("done")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "done" in r.stdout, (r.returncode, r.stderr[-500:])


def _scratch_bound(fmt, m, n, d, terms):
    """The activation operands (lane records of 16 bytes MXFP4, 48 bytes HiF4, one scale byte each) and
    the K-split partial tiles of 64 x 128 outputs in up to four splits, 256-byte aligned."""
    def al(x):
        return -(-x // 256) * 256
    lanes = -(-m // 32) * -(-d // 64) * 64
    tiles = -(-m // 64) * -(-n // 128)
    return terms * (al(lanes * (16 if fmt == "mxfp4" else 48)) + al(lanes)) + tiles * min(4, 256 // tiles) * 64 * 128 * 4


@pytest.mark.parametrize("fmt", ["mxfp4", "hif4"])
@pytest.mark.parametrize("sp,terms", [("none", 1), ("2:4", 2)])
def test_streamed_splits_keep_the_scratch_bound(fmt, sp, terms):
    """A K split of the 32-row tiles takes no more scratch than one of 64 x 128 tiles in four
    splits: calls at the limit of the library's own scratch stay accepted."""
    for m, n, d in itertools.product((1, 8, 32, 33, 64, 65, 96, 97, 128, 160, 200, 229, 256), (1, 32, 33, 64, 96, 113, 256, 400, 510),
                                     (32768, 40960, 65536, 131072)):
        if P.gemm_plan(fmt, m, n, d)["ksplit"] == 1:
            continue
        need = P.resq_workspace_size(P.OP_LINEAR_FWD_PREPARED, P.FORMATS[fmt], P.sparsity_code(sp), m, d, n)
        assert need <= _scratch_bound(fmt, m, n, d, terms), (m, n, d, need)


def test_noalloc_limit_is_not_passed_by_a_split():
    """Forward calls that fit the library's scratch with the 64 x 128 tiles' partials."""
    for m, d, n in ((97, 350528, 96), (97, 350528, 128), (98, 348096, 256)):
        need = P.resq_workspace_size(P.OP_LINEAR_FWD_PREPARED, P.FORMATS["mxfp4"], P.sparsity_code("unstructured50"), m, d, n)
        assert need <= P.NOALLOC_SCRATCH_BYTES, (m, d, n, need)
