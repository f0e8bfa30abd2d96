"""A device without room for the matrix-core kernels' own copy of the bootstrapping key still takes
the key set: the other kernels run, with the oracle's bits.  The second allocation of the key's
size fails by a hipMalloc in front of the runtime's, in a process of its own."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes as C, sys
shim = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)  # before the library, so that its hipMalloc is this one
import numpy as np
import oracle
from paper_2310_12441_amd import binding
from synth import Params, Q2_DEFAULT, enc_draws, key_draws, messages, negacyclic_table
C.c_void_p.in_dll(shim, "real_malloc").value = C.cast(binding.lib.hipMalloc, C.c_void_p).value
size, after, failed = (t.in_dll(shim, n) for t, n in ((C.c_size_t, "fail_bytes"), (C.c_int, "fail_after"), (C.c_int, "failed")))
for p in (Params(n=5, N=1024, log2_B=7, l=4), Params(n=3, N=2048, log2_B=15, l=4, Q2=Q2_DEFAULT, ternary=True)):
    draws = key_draws(p, 3300)
    primes = 2 if p.Q2 else 1
    size.value, after.value, failed.value = p.n * p.keys_per_coord * 2 * p.l * 2 * p.N * 4 * primes, 1, 0
    ctx = binding.Context(p, draws)
    ctx.device_init(0)
    assert failed.value == 1, failed.value
    size.value = 0
    r, t = 4, 64
    q, f = 2 * p.N * r, negacyclic_table(t, t, 60)
    keys = (oracle.KeySetWide if p.Q2 else oracle.KeySet)(p, draws)
    V = oracle.w_test_vector(p.N, r, p.Q_ring, t, t, f) if p.Q2 else oracle.test_vector(p.N, r, p.Q, t, t, f)
    ed = enc_draws(p.n, q, 3, 70)
    ct = oracle.encrypt(p.n, q, t, keys.s, messages(t, 3, 80), ed["a"], ed["e"])
    want = (oracle.w_bootstrap_many if p.Q2 else oracle.bootstrap_many)(p, r, keys.bsk, keys.ksk, V, q, q, ct)
    tid = ctx.table_create(t, t, r, f)
    for count in (3, 300):
        pick = np.arange(count) % 3
        np.testing.assert_array_equal(ctx.bootstrap([tid] * count, ct[pick]), want[pick])
    if not p.Q2:
        x = np.random.default_rng(1).integers(0, p.Q, (2, 2, p.N), dtype=np.uint32)
        np.testing.assert_array_equal(ctx.external_product(1, x)[1], oracle.external_product(keys.bsk[1], x[1], p.Q, 7, 4))
        np.testing.assert_array_equal(ctx.negacyclic_mul(x[0], x[1])[1], oracle.poly_mul(x[0, 1], x[1, 1], p.Q))
    ctx.close()
    print("N", p.N, "without the second key: exact", flush=True)
"""


def test_key_set_without_room_for_a_second_copy(tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    shim = str(tmp_path / "fail_malloc.so")
    subprocess.run(["gcc", "-shared", "-fPIC", os.path.join(ROOT, "tests", "c", "fail_malloc.c"), "-o", shim], check=True)
    res = subprocess.run([sys.executable, "-c", CHILD, shim], capture_output=True, text=True, timeout=100, cwd=ROOT)
    print(res.stdout, res.stderr[-2000:])
    assert res.returncode == 0 and res.stdout.count("exact") == 2
