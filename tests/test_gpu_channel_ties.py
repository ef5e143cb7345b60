"""Channel selection with many equal keys: the ways through the top-k that ordinary keys do not take.
Rows are constant within a 64-column block, so a block's 64 channels share one key; blocks of two
kinds differ in one row of tiny values, i.e. only in key bits below the 32 that the top-k holds in
LDS.  What each case is meant to reach is asserted on the CPU from the oracle's keys; masks equal the
oracle's bit for bit."""
import numpy as np
import pytest

from oracle import resq as Q
from synth import bf16_bits_to_f32, f32_to_bf16_bits
from _gpu_util import log

FMTS = ["mxfp4", "hif4"]
LOW = 31        # key bits below the upper 32 (the sign excluded)
GATHER = 1024   # keys that the top-k gathers, one per thread
# kind: blocks without and with the tiny row, blocks of distinct larger values, blocks of zeros
CASES = {
    "one_key": (30, 0, 3, 0),           # more than 1024 ties, and low bits
    "lower_of_two": (24, 16, 0, 0),     # threshold below keys that differ in low bits alone
    "upper_of_two": (16, 24, 0, 0),     # threshold above such keys
    "gathered_lower": (9, 6, 0, 0),     # the same with at most 1024 keys sharing the upper bits
    "gathered_upper": (5, 9, 1, 0),
    "zeros_1088": (2, 2, 2, 11),        # threshold 0 below nonzero keys, items past n among the zeros
    "zeros_2112": (4, 6, 3, 20),
}


def _x(kind, m):
    a, b, big, zero = CASES[kind]
    rng = np.random.default_rng([m, *map(ord, kind)])
    rows = (rng.standard_normal(m) * np.exp2(rng.integers(0, 6, m))).astype(np.float32)
    tiny = int(rng.integers(0, m))
    cols = []
    for _ in range(a):
        cols.append(rows.copy())
        cols[-1][tiny] = 0.0
    for _ in range(b):
        cols.append(rows.copy())
        cols[-1][tiny] = 1.2109375 * 2.0 ** -14
    for i in range(big):
        cols.append(rows * np.float32(1.375 + i))
    cols += [np.zeros(m, np.float32)] * zero
    order = rng.permutation(len(cols))
    return f32_to_bf16_bits(np.repeat(np.stack([cols[i] for i in order], 1), 64, axis=1))


@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("kind", list(CASES))
@pytest.mark.parametrize("m", [129, 260])
def test_the_cases_are_what_they_are_meant_to_be(fmt, kind, m):
    bits = _x(kind, m)
    d = bits.shape[1]
    keys = Q.channel_keys(Q.resq_quantize_residual(fmt, "identity", bf16_bits_to_f32(bits))["srhat"]).view(np.uint64)
    keep = d // 2
    T = np.sort(keys)[::-1][keep - 1]
    upper = keys >> np.uint64(LOW)
    same_upper, ties, above = (int((c).sum()) for c in (upper == T >> np.uint64(LOW), keys == T, keys > T))
    assert ties > keep - above > 0, "some of the ties are kept, not all: they are ranked by index"
    if kind.startswith("zeros"):
        assert T == 0 and 0 < above < keep and d % GATHER != 0
        return
    assert (keys & np.uint64((1 << LOW) - 1)).any(), "low bits count"
    assert ties > 64, "more than one wave ranks directly"
    assert (same_upper > GATHER) == (not kind.startswith("gathered"))
    sharing = keys[upper == T >> np.uint64(LOW)]
    if kind.endswith("lower") or kind.startswith("lower"):
        assert (sharing > T).any() and not (sharing < T).any()
    elif kind.endswith("upper") or kind.startswith("upper"):
        assert (sharing < T).any() and not (sharing > T).any()
    else:
        assert same_upper == ties


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", FMTS)
@pytest.mark.parametrize("kind", list(CASES))
@pytest.mark.parametrize("m", [129, 260])
def test_tied_channels(fmt, kind, m):
    from test_gpu_select import _check_select
    bits = _x(kind, m)
    log(f"tied channels {fmt} {kind} {m}x{bits.shape[1]}")
    _check_select(fmt, "channel50", bits)
