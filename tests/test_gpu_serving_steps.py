"""Serving by one launch per step: ticks whose chunk does not divide n, so that ciphertexts end inside
a tick and are carried over beside others that go on, exact against the oracle."""
import numpy as np
import pytest

from gpu_setup import Setup
from synth import Params, Q2_DEFAULT

pytestmark = pytest.mark.gpu


def _served(s, rs, arrivals):
    ids, cts, want = s.batch(rs)
    srv = s.ctx.server_start(256 << 20, chunk_steps=3)
    try:
        print("serving N", s.p.N, "requests", len(rs), flush=True)
        out, lat = srv.replay(ids, cts, arrivals)
    finally:
        srv.stop()
    assert np.all(lat > 0)
    np.testing.assert_array_equal(out, want)


@pytest.mark.parametrize("ternary", [False, True])
def test_bursts_at_1024(ternary):
    """Bursts of r = 8 on the two digit groups, and past two components per compute unit on the fused
    kernel; up to sixteen that end together are key-switched by the i-split kernel, more by lanes."""
    s = Setup(Params(n=7, N=1024, log2_B=7, l=4, ternary=ternary), 3200 + ternary)
    for count in (1, 16, 17, 64, 70):
        _served(s, [8] * count, np.zeros(count, np.int64))
    s.ctx.close()


@pytest.mark.parametrize("ternary", [False, True])
def test_two_primes_at_2048(ternary):
    """Few components (one workgroup per component and prime) and more than 3/2 per compute unit (two
    components per workgroup), arriving over several ticks, so that a workgroup's two components may stand
    at different steps."""
    s = Setup(Params(n=7, N=2048, log2_B=15, l=4, Q2=Q2_DEFAULT, ternary=ternary), 3210 + ternary)
    _served(s, [2, 1, 5], np.zeros(3, np.int64))
    _served(s, [3] * 320, np.arange(320) // 4 * 20_000)
    s.ctx.close()
