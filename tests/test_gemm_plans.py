"""The GEMM's plans, as the host-side query reports them (CPU)."""
import itertools

import pytest

import paper_2607_26515_amd as P


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
