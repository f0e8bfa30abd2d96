"""The key switch with one ciphertext per lane at the edges of its column groups (64 and 128
samples) and of its splits, with a full tile of rows and a partial one, against the oracle."""
import numpy as np
import pytest

import oracle
from synth import Params, key_draws

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("log2_Bks,l_ks", [(4, 8), (1, 31)])
def test_column_groups(log2_Bks, l_ks):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_12441_amd import binding
    p = Params(n=70, N=256, log2_B=8, l=3, log2_Bks=log2_Bks, l_ks=l_ks)
    draws = key_draws(p, 2500)
    ctx, keys = binding.Context(p, draws), oracle.KeySet(p, draws)
    ctx.device_init(0)
    lwe = np.random.default_rng(7).integers(0, p.Q, size=(257, p.N + 1), dtype=np.uint32)
    lwe[3, :] = p.Q - 1
    want = np.array([oracle.keyswitch(p, keys.ksk, x) for x in lwe])
    for count in (1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257):
        print("key switch base 2^%d, %d samples" % (log2_Bks, count), flush=True)
        np.testing.assert_array_equal(ctx.keyswitch(lwe[:count]), want[:count], err_msg=f"{count} samples")
    ctx.close()
