"""Schedules of the per-step path name the kernel that runs: at N = 1024 the matrix-core step (one
wave per component), the butterfly step of four waves and its two digit groups are three different
schedules, the defaults say which of them they take, and every one gives the oracle's bits."""
from dataclasses import replace

import numpy as np
import pytest

from gpu_setup import Setup
from synth import Params, Q2_DEFAULT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ternary", [False, True])
def test_per_step_schedules_at_1024(ternary):
    s = Setup(replace(Params(n=4, N=1024, log2_B=7, l=4), ternary=ternary), 3100 + ternary)
    step, four, groups = (0, 1, 0), (0, 4, 0), (0, 4, 4)
    # tables the fused kernel holds: all three are candidates
    ids, cts, want = s.batch([4] * 40)
    shapes = s.shapes(ids)
    assert {k for k in shapes if k[0] == 0} == {step, four, groups}
    for shape in (step, four, groups):
        s.ctx.set_schedule(ids, shapes[shape])
        assert s.default(ids) == shape
        np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want, err_msg=str(shape))
    # wider tables: the digit groups up to 3/2 components per compute unit, the step above
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for count in (1, 3 * cus // 32, 3 * cus // 32 + 1):
        ids, cts, want = s.batch([16] * count)
        light = 2 * 16 * count <= 3 * cus
        assert s.default(ids) == (groups if light else step), count
        acc = s.ctx.blind_rotate(ids[:1], cts[:1], s.p.n)  # a batch of its own: light
        for shape, k in s.shapes(ids).items():
            assert shape in (step, groups)
            s.ctx.set_schedule(ids, k)
            np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want, err_msg=f"{count} {shape}")
            if count == 1:
                np.testing.assert_array_equal(s.ctx.blind_rotate(ids, cts, s.p.n), acc)
    s.ctx.close()


def test_key_switch_behind_steps():
    """Up to 16 ciphertexts at one prime and N = 1024 the i-split key switch, which spares the cached
    bootstrapping key; at two primes, whose key no cache keeps, the one by lanes."""
    for p, few in ((Params(n=4, N=1024, log2_B=7, l=4), 0), (Params(n=4, N=2048, log2_B=15, l=4, Q2=Q2_DEFAULT), 2)):
        s = Setup(p, 3150 + few)
        for count, kernel in ((1, few), (16, few), (17, 2)):
            ids, cts, want = s.batch([8] * count)
            assert s.ctx.schedule_describe(ids)[4] == kernel, (p.N, count)
            np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want, err_msg=f"{p.N} {count}")
        s.ctx.close()
