"""A context on the GPU beside the oracle's keys, with batches and their expected outputs."""
import numpy as np
import pytest

import oracle
from synth import enc_draws, key_draws, messages, negacyclic_table


def _binding():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_12441_amd import binding
    return binding


class Setup:
    """A context, its oracle keys, and ciphertexts of tables of t = 64 with their oracle results."""

    def __init__(self, p, seed):
        draws = key_draws(p, seed)
        self.p = p
        self.ctx = _binding().Context(p, draws)
        self.ctx.device_init(0)
        self.keys = (oracle.KeySetWide if p.Q2 else oracle.KeySet)(p, draws)
        self.tabs = {}

    def batch(self, rs, distinct=4):
        """ids, ciphertexts and the oracle's outputs for components rs (the first `distinct` of
        each r are drawn, the rest repeat them)."""
        p, made, ids, cts, want = self.p, {}, [], [], []
        for j, r in enumerate(rs):
            have = made.setdefault(r, [])
            if len(have) < distinct:
                q = 2 * p.N * r
                if r not in self.tabs:
                    self.tabs[r] = self.ctx.table_create(64, 64, r, negacyclic_table(64, 64, 60 + r))
                ed = enc_draws(p.n, q, 1, 900 + j)
                ct = oracle.encrypt(p.n, q, 64, self.keys.s, messages(64, 1, 800 + j), ed["a"], ed["e"])
                f = negacyclic_table(64, 64, 60 + r)
                if p.Q2:
                    w = oracle.w_bootstrap_many(p, r, self.keys.bsk, self.keys.ksk,
                                                oracle.w_test_vector(p.N, r, p.Q_ring, 64, 64, f), q, q, ct)
                else:
                    w = oracle.bootstrap_many(p, r, self.keys.bsk, self.keys.ksk,
                                              oracle.test_vector(p.N, r, p.Q, 64, 64, f), q, q, ct)
                have.append((ct[0], w[0]))
            ct, w = have[j % len(have)]
            ids.append(self.tabs[r])
            cts.append(ct)
            want.append(w)
        return np.array(ids, np.int32), np.array(cts), np.array(want)

    def shapes(self, ids):
        """(group waves, waves per component, NTT schedule) -> first choice of that shape."""
        out = {}
        for k in range(self.ctx.schedule_count(ids)):
            d = self.ctx.schedule_describe(ids, k)
            out.setdefault((d[0], d[3], d[5]), k)
        return out

    def default(self, ids):
        d = self.ctx.schedule_describe(ids)
        return d[0], d[3], d[5]
