"""The blind rotation on the matrix cores (N = 1024, digits of at most 7 bits), exact
against the oracle: every gadget length and digit width at the edges of its range, both
secrets, r from 1 to 8 in groups with idle component slots, one CMux step and many, and
keys whose NTT values all sit at the largest magnitude a residue can have."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
from synth import Q2_DEFAULT, Params, enc_draws, key_draws, messages, negacyclic_table

pytestmark = pytest.mark.gpu
N = 1024


def _binding():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_12441_amd import binding
    return binding


def _context(p, seed, draws=None):
    draws = draws or key_draws(p, seed)
    ctx = _binding().Context(p, draws)
    ctx.device_init(0)
    return ctx, oracle.KeySet(p, draws)


def _fused(ctx, ids, waves=1):
    """Pin the fused shape with `waves` waves per component, lockstep schedule."""
    for k in range(ctx.schedule_count(ids)):
        d = ctx.schedule_describe(ids, k)
        if d[0] == 8 and d[3] == waves and d[5] == 0:
            return ctx.set_schedule(ids, k)
    raise AssertionError("no fused schedule")


@pytest.mark.parametrize("l,log2_B,ternary,Q", [(1, 7, False, 0), (2, 7, True, 0), (3, 7, False, 0), (4, 7, True, 0),
                                                (4, 1, False, 0), (4, 5, True, 0), (4, 7, False, 12289),
                                                (4, 6, False, 1073692673)])
def test_fused_steps_and_bootstrap(l, log2_B, ternary, Q):
    p = replace(Params(n=6, N=N, log2_B=log2_B, l=l), ternary=ternary)
    if Q:
        p = replace(p, Q=Q)
    ctx, keys = _context(p, 2100 + 10 * l + log2_B)
    ids, cts, Vs, rs = [], [], [], []
    for k, r in enumerate((1, 8, 3, 2, 5)):
        t = 64
        f = negacyclic_table(t, 64, 60 + k)
        tid = ctx.table_create(t, 64, r, f, 2 * N * r if r in (1, 2, 8) else 12289)
        q = 2 * N * r if r in (1, 2, 8) else 12289
        ed = enc_draws(p.n, q, 1, 70 + k)
        ids.append(tid)
        cts.append(oracle.encrypt(p.n, q, t, keys.s, messages(t, 1, 80 + k), ed["a"], ed["e"])[0])
        Vs.append(oracle.test_vector(N, r, p.Q, t, 64, f))
        rs.append((r, q))
    print("matrix core l", l, "log2_B", log2_B, "ternary", ternary, "Q", p.Q, flush=True)
    for steps in (1, p.n):
        got, off = ctx.blind_rotate(ids, np.array(cts), steps), 0
        for j, (r, q) in enumerate(rs):
            size = r * 2 * N
            want = oracle.blind_rotate(p, r, keys.bsk, Vs[j], oracle.modswitch(cts[j], q, 2 * N * r), steps)
            np.testing.assert_array_equal(got[off:off + size].reshape(r, 2, N), want, err_msg=f"r {r} steps {steps}")
            off += size
    _fused(ctx, ids)
    out = ctx.bootstrap(ids, np.array(cts), q_out=p.Q)
    for j, (r, q) in enumerate(rs):
        np.testing.assert_array_equal(out[j], oracle.bootstrap(p, r, keys.bsk, keys.ksk, Vs[j], q, p.Q, cts[j]))
    # two waves per component: r <= 4, with idle slots, and more groups than compute units
    narrow = [j for j, (r, _) in enumerate(rs) if r <= 4] * 200
    _fused(ctx, [ids[j] for j in narrow], 2)
    np.testing.assert_array_equal(ctx.bootstrap([ids[j] for j in narrow], np.array(cts)[narrow], q_out=p.Q), out[narrow])
    ctx.close()


@pytest.mark.parametrize("sign", [1, -1])
def test_largest_key_magnitude(sign):
    """Masks a(x) = c with c 2^64 / N = +-(Q - 1) / 2: every NTT value the products read on that
    side is the largest balanced residue, so the 64-bit sums come as near their bound as keys can
    bring them."""
    p = Params(n=3, N=N, log2_B=7, l=4)
    draws = key_draws(p, 2200)
    c = sign * (p.Q - 1) // 2 * N * pow(pow(2, 64, p.Q), p.Q - 2, p.Q) % p.Q
    draws["bsk_a"] = np.zeros_like(draws["bsk_a"])
    draws["bsk_a"][:, :, 0] = c
    ctx, keys = _context(p, 0, draws)
    r, t = 4, 64
    f = negacyclic_table(t, 64, 61)
    tid = ctx.table_create(t, 64, r, f)
    V = oracle.test_vector(N, r, p.Q, t, 64, f)
    ed = enc_draws(p.n, 2 * N * r, 2, 71)
    ct = oracle.encrypt(p.n, 2 * N * r, t, keys.s, messages(t, 2, 81), ed["a"], ed["e"])
    got = ctx.blind_rotate([tid] * 2, ct, 3).reshape(2, r, 2, N)
    for j in range(2):
        np.testing.assert_array_equal(got[j], oracle.blind_rotate(p, r, keys.bsk, V, ct[j], 3))
    ctx.close()


@pytest.mark.parametrize("count", [257, 513, 700])
def test_rounds_with_a_thin_tail(count):
    """Batches whose last round of groups is spread over all compute units equal the same
    ciphertexts one by one (r = 8: one ciphertext per full group, so 256 fill a round)."""
    p = Params(n=5, N=N, log2_B=7, l=4)
    ctx, keys = _context(p, 2300)
    tabs = [(r, ctx.table_create(64, 64, r, negacyclic_table(64, 64, 90 + r))) for r in (8, 1, 4)]
    pick = [tabs[0] if j < 256 else tabs[j % 3] for j in range(count)]
    cts = np.array([oracle.encrypt(p.n, 2 * N * r, 64, keys.s, messages(64, 1, j), *(lambda e: (e["a"], e["e"]))(
        enc_draws(p.n, 2 * N * r, 1, j)))[0] for j, (r, _) in enumerate(pick)])
    ids = np.array([tid for _, tid in pick], np.int32)
    _fused(ctx, ids)
    np.testing.assert_array_equal(ctx.bootstrap(ids, cts), ctx.bootstrap(ids, cts, plain=True))
    ctx.close()


@pytest.mark.parametrize("l,log2_B,ternary", [(4, 15, False), (4, 15, True), (3, 15, True), (1, 15, False), (2, 7, False),
                                              (4, 1, True)])
def test_two_primes_2048(l, log2_B, ternary):
    """The 54-bit ring modulus at N = 2048: odd and even gadget lengths, digit widths at both
    ends, r from 1 to 3 with an odd number of components (a workgroup holds two), against the
    oracle's uint64 statement; then a batch of more components than one round of workgroups
    holds equals its ciphertexts in other shapes."""
    p = Params(n=4, N=2048, log2_B=log2_B, l=l, Q2=Q2_DEFAULT, ternary=ternary)
    draws = key_draws(p, 2400 + 10 * l + log2_B)
    ctx, keys = _binding().Context(p, draws), oracle.KeySetWide(p, draws)
    ctx.device_init(0)
    print("two primes l", l, "log2_B", log2_B, "ternary", ternary, flush=True)
    ids, cts, Vs, rs = [], [], [], []
    for k, r in enumerate((1, 3, 1)):
        f = negacyclic_table(32, 32, 60 + k)
        q = 2 * 2048 * r
        ed = enc_draws(p.n, q, 1, 70 + k)
        ids.append(ctx.table_create(32, 32, r, f))
        cts.append(oracle.encrypt(p.n, q, 32, keys.s, messages(32, 1, 80 + k), ed["a"], ed["e"])[0])
        Vs.append(oracle.w_test_vector(2048, r, p.Q_ring, 32, 32, f))
        rs.append(r)
    got, off = ctx.blind_rotate(ids, np.array(cts), p.n), 0
    for r, V, ct in zip(rs, Vs, cts):
        np.testing.assert_array_equal(got[off:off + r * 4096].reshape(r, 2, 2048),
                                      oracle.w_blind_rotate(p, r, keys.bsk, V, ct, p.n), err_msg=f"r {r}")
        off += r * 4096
    ids, cts = np.array([ids[j % 3] for j in range(601)], np.int32), np.array([cts[j % 3] for j in range(601)])
    shapes = {ctx.schedule_describe(ids, k)[5]: k for k in reversed(range(ctx.schedule_count(ids)))}
    ctx.set_schedule(ids, shapes[0])
    out = ctx.bootstrap(ids, cts)
    ctx.set_schedule(ids, shapes[5])
    np.testing.assert_array_equal(ctx.bootstrap(ids, cts), out)
    ctx.close()


@pytest.mark.parametrize("l,log2_B,ternary,Q", [(1, 7, False, 0), (3, 6, True, 0), (4, 7, False, 0), (4, 7, True, 12289)])
def test_external_products(l, log2_B, ternary, Q):
    """One external product per pair of waves and per wave (more than four per compute unit),
    with part-filled workgroups at the end, and the coefficients where rounding and centring turn."""
    p = replace(Params(n=2, N=N, log2_B=log2_B, l=l), ternary=ternary)
    if Q:
        p = replace(p, Q=Q)
    ctx, keys = _context(p, 2500 + l)
    rng = np.random.default_rng(l)
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    pairs = rng.integers(0, p.Q, (4 * cus + 9, 2, N), dtype=np.uint32)
    edges = np.array([0, 1, p.Q // 2 - 1, p.Q // 2, p.Q // 2 + 1, p.Q - 2, p.Q - 1], np.uint32)
    pairs[0] = edges[rng.integers(0, len(edges), (2, N))]
    pairs[-1] = p.Q // 2
    i = len(keys.bsk) - 1
    for count in (1, 7, len(pairs)):
        sub = pairs[-count:].copy()
        sub[0] = pairs[0]
        got = ctx.external_product(i, sub)
        for k in {0, count // 2, count - 1}:
            np.testing.assert_array_equal(got[k], oracle.external_product(keys.bsk[i], sub[k], p.Q, log2_B, l),
                                          err_msg=f"count {count} item {k}")
    ctx.close()


@pytest.mark.parametrize("Q", [0, 12289, 1073692673])
def test_ring_products(Q):
    """Products of polynomials of full-width residues: edges of the centred range, part-filled
    workgroups, and more products than the grid holds at once."""
    p = Params(n=2, N=N, log2_B=6 if Q else 7, l=4)
    if Q:
        p = replace(p, Q=Q)
    ctx, _ = _context(p, 2600)
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(p.Q)
    a, b = rng.integers(0, p.Q, (2, 12 * cus + 5, N), dtype=np.uint32)
    edges = np.array([0, 1, p.Q // 2, p.Q // 2 + 1, p.Q - 1], np.uint32)
    a[0], b[0] = edges[rng.integers(0, len(edges), (2, N))]
    a[-1], b[-1] = p.Q // 2, p.Q - 1
    a[-2], b[-2] = p.Q // 2 + 1, p.Q // 2 + 1
    for count in (1, 6, len(a)):
        x, y = a[-count:].copy(), b[-count:].copy()
        x[0], y[0] = a[0], b[0]
        got = ctx.negacyclic_mul(x, y)
        for k in {0, count // 2, max(0, count - 2), count - 1}:
            np.testing.assert_array_equal(got[k], oracle.poly_mul(x[k], y[k], p.Q), err_msg=f"count {count} item {k}")
    ctx.close()


@pytest.mark.parametrize("rs,count", [((1,), 3), ((1,), 300), ((1, 2, 3), 200)])
def test_spread_groups(rs, count):
    """Batches light enough for one or two components per group, an odd remainder and
    ciphertexts wider than the group's share among them, equal the same one by one."""
    p = Params(n=4, N=N, log2_B=7, l=4)
    ctx, keys = _context(p, 2700)
    tabs = [(r, ctx.table_create(64, 64, r, negacyclic_table(64, 64, 95 + r), 2 * N * 6)) for r in rs]
    pick = [tabs[j % len(tabs)] for j in range(count)]
    ed = enc_draws(p.n, 2 * N * 6, count, 9)
    cts = oracle.encrypt(p.n, 2 * N * 6, 64, keys.s, messages(64, count, 8), ed["a"], ed["e"])
    ids = np.array([tid for _, tid in pick], np.int32)
    _fused(ctx, ids, 2)
    np.testing.assert_array_equal(ctx.bootstrap(ids, cts), ctx.bootstrap(ids, cts, plain=True))
    ctx.close()
