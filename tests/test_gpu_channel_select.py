"""Channel selection where its kernels can go wrong: channel counts at the edges of the key
kernel's 64-channel workgroups, of the top-k's 1024-key slots and of the keys that fit its LDS
(20480; more are streamed); row counts at the edges of the 128-row steps and the four steps
loaded together; and keys that are all tied, few and distinct, zero for some blocks or far apart.
Hundreds to thousands of ties at the threshold are test_gpu_channel_ties.py's.  Masks equal the
oracle's bit for bit."""
import numpy as np
import pytest

from synth import f32_to_bf16_bits
from _gpu_util import log
from test_gpu_select import _check_select

pytestmark = pytest.mark.gpu

KINDS = ["spread", "few_values", "zero_half", "mostly_tied", "wide"]


def _x(kind, m, d, rng):
    x = rng.standard_normal((m, d)).astype(np.float32)
    if kind == "few_values":  # every scale block the same: at most 64 distinct keys
        x = np.tile(x[:, :64], (1, d // 64))
    elif kind == "zero_half":  # whole scale blocks of zeros
        x[:, np.repeat(rng.random(d // 64) < 0.45, 64)] = 0.0
    elif kind == "mostly_tied":  # equal scale blocks, a few of them scaled up or down
        x = np.tile(x[:, :64], (1, d // 64))
        x *= np.repeat(np.where(rng.random(d // 64) < 0.1, 2.0 ** rng.integers(-3, 4, d // 64), 1.0), 64)
    elif kind == "wide":
        x *= np.exp2(rng.integers(-30, 30, d // 64)).astype(np.float32).repeat(64)
        x *= np.exp2(rng.integers(0, 12, (m, 1))).astype(np.float32)
    return f32_to_bf16_bits(x.astype(np.float32))


@pytest.mark.parametrize("fmt", ["mxfp4", "hif4"])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("m,d", [(1, 1024), (127, 1088), (129, 64), (511, 192), (513, 2112),
                                 (7, 20480), (3, 20544)])
def test_channel_select_edges(fmt, kind, m, d):
    log(f"channel select {fmt} {kind} {m}x{d}")
    rng = np.random.default_rng([m, d, KINDS.index(kind)])
    _check_select(fmt, "channel50", _x(kind, m, d, rng))
