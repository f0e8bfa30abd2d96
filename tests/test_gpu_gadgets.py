"""Every kernel a gadget leads to, exact against the oracle: the butterfly kernels that run where
the matrix-core kernels do not apply (digits of more than 7 bits or a gadget longer than four at
N = 1024, longer than four at N = 2048 with two primes), and the matrix-core step and the
workgroups per prime at each gadget length."""
import numpy as np
import pytest

import oracle
from gpu_setup import Setup
from synth import Params, Q2_DEFAULT

pytestmark = pytest.mark.gpu


def _each_shape(s, rs):
    """Every blind-rotation shape of a batch of components rs gives the oracle's bits; the shapes."""
    ids, cts, want = s.batch(rs)
    shapes = s.shapes(ids)
    np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want, err_msg="default")
    for shape, k in shapes.items():
        print("  ", len(rs), "ciphertexts, shape", shape, flush=True)
        s.ctx.set_schedule(ids, k)
        np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want, err_msg=str(shape))
    return set(shapes)


@pytest.mark.parametrize("ternary", [False, True])
@pytest.mark.parametrize("l,log2_B", [(3, 10), (5, 6)])
def test_butterflies_at_1024(l, log2_B, ternary):
    p = Params(n=4, N=1024, log2_B=log2_B, l=l, ternary=ternary)
    s = Setup(p, 3400 + 10 * l + ternary)
    print("butterflies l", l, "log2_B", log2_B, "ternary", ternary, flush=True)
    # group waves, waves per component, schedule: lockstep (2) and the per-step shapes among them
    assert _each_shape(s, [4, 1, 3] * 14) >= {(8, 1, 0), (4, 1, 0), (8, 2, 0), (8, 1, 2), (4, 1, 2), (0, 2, 0), (0, 4, 0),
                                             (0, 4, 4)}
    assert _each_shape(s, [8] * 5) >= {(8, 1, 0), (8, 1, 2), (0, 2, 0), (0, 4, 0), (0, 4, 4)}
    _each_shape(s, [12] * 3)
    x = np.random.default_rng(l).integers(0, p.Q, (2, 5, 2, p.N), dtype=np.uint32)
    i = p.n * p.keys_per_coord - 1
    got = s.ctx.external_product(i, x[0])
    prod = s.ctx.negacyclic_mul(x[0, :, 0], x[1, :, 0])
    for k in range(5):
        np.testing.assert_array_equal(got[k], oracle.external_product(s.keys.bsk[i], x[0, k], p.Q, log2_B, l))
        np.testing.assert_array_equal(prod[k], oracle.poly_mul(x[0, k, 0], x[1, k, 0], p.Q))
    s.ctx.close()


@pytest.mark.parametrize("l,log2_B", [(1, 7), (2, 7), (3, 7), (4, 7), (4, 1)])
@pytest.mark.parametrize("ternary", [False, True])
def test_step_at_1024(l, log2_B, ternary):
    """Batches of r > 8 above and below 3/2 components per compute unit, the last workgroup part-filled."""
    s = Setup(Params(n=4, N=1024, log2_B=log2_B, l=l, ternary=ternary), 3500 + 10 * l + log2_B + ternary)
    import torch
    heavy = 3 * torch.cuda.get_device_properties(0).multi_processor_count // 32 + 1
    print("matrix-core step l", l, "log2_B", log2_B, "ternary", ternary, flush=True)
    for rs in ([16] * heavy + [9], [9, 16, 11]):
        ids, _, _ = s.batch(rs)
        assert s.default(ids) == ((0, 1, 0) if len(rs) > 3 else (0, 4, 4))
        assert _each_shape(s, rs) == {(0, 1, 0), (0, 4, 4)}
    s.ctx.close()


@pytest.mark.parametrize("l,log2_B,ternary", [(1, 15, False), (1, 7, True), (2, 15, True), (2, 7, False), (3, 15, False),
                                              (3, 15, True), (4, 15, False), (4, 1, True), (5, 10, False), (5, 10, True)])
def test_two_primes_at_2048(l, log2_B, ternary):
    """One workgroup per component, and per component and prime, of one and two digit groups; l > 4: butterflies."""
    s = Setup(Params(n=4, N=2048, log2_B=log2_B, l=l, Q2=Q2_DEFAULT, ternary=ternary), 3600 + 10 * l + log2_B + ternary)
    print("two primes l", l, "log2_B", log2_B, "ternary", ternary, flush=True)
    assert {k[2] for k in _each_shape(s, [1, 3, 1, 2])} == {0, 5, 6}
    s.ctx.close()


@pytest.mark.parametrize("l,ternary,shapes", [(1, True, (6, 5, 5)), (2, False, (6, 5, 0)), (3, True, (6, 6, 0)), (4, False, (6, 6, 0))])
def test_two_primes_at_2048_by_count(l, ternary, shapes):
    """Up to one component for every two compute units, up to 3/2 per unit, and more: the untuned shape of
    each, bootstraps against the oracle and blind rotations against the same ciphertexts in a small batch."""
    s = Setup(Params(n=3, N=2048, log2_B=15, l=l, Q2=Q2_DEFAULT, ternary=ternary), 3700 + 10 * l + ternary)
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    few = s.ctx.blind_rotate(*s.batch([2] * 4)[:2], s.p.n).reshape(4, -1)
    for count, shape in zip((cus // 4, cus // 4 + 1, cus * 3 // 4 + 1), shapes):
        ids, cts, want = s.batch([2] * count)
        print("two primes l", l, "ternary", ternary, "components", 2 * count, "shape", shape, flush=True)
        assert s.default(ids)[2] == shape
        np.testing.assert_array_equal(s.ctx.bootstrap(ids, cts), want)
        acc = s.ctx.blind_rotate(ids, cts, s.p.n).reshape(count, -1)
        np.testing.assert_array_equal(acc, few[np.arange(count) % 4])
    s.ctx.close()
