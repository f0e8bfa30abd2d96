"""The work that a program has this library do, as measurable cases.

A case names a key set (one of the parameter sets of ``synth.PRESETS`` or the
ternary variant of the paper-shaped one), an entry point, the tables its
ciphertexts evaluate and a count.  A key set outlives every batch in a real
program, so a key set (its Context) is made once per process and kept; the
ciphertexts, samples and polynomials are drawn from the case's seed.
"""
from __future__ import annotations

from dataclasses import replace
from functools import lru_cache
import math

import numpy as np
import torch

from paper_2310_12441_amd import binding
from synth import PRESETS, enc_draws, key_draws, messages, negacyclic_table

KEY_SEED = 1
_PAPER = PRESETS["paper_shaped"]["params"]
KEY_SETS = {
    "paper": _PAPER,                                   # n = 630, N = 1024, gadget 2^7 x 4
    "ternary": replace(_PAPER, ternary=True),          # the same with two RGSW keys per coordinate
    "tfhe": PRESETS["tfhe_shaped"]["params"],          # one ring of N = 4096
    "margin": PRESETS["paper_margin"]["params"],       # N = 2048, 54-bit ring modulus, ternary
}
# plaintext size of a table of r components: the (t, r) classes of the uneven batch
# and of the serving trace at N = 1024 and their continuation, t = 2^12 on the ring of
# 4096, and 2Nr / t = 128 at the paper-margin parameters
PLAIN_N1024 = {1: 256, 2: 1024, 4: 4096, 8: 16384, 16: 32768, 32: 65536}


def plaintext_size(keys: str, r: int) -> int:
    if keys == "tfhe":
        return 4096 * r
    return 32 * r if keys == "margin" else PLAIN_N1024[r]


def listed():
    return [
        # an interactive caller: one ciphertext in host memory, by the unbatched path
        dict(name="plain_one", op="bootstrap", keys="paper", r="4", count=1, general=False, plain=True, host=True),
        # a small service tick, odd count, buffers on the device
        dict(name="batch_37", op="bootstrap", keys="paper", r="4", count=37, general=False, plain=False, host=False),
        # the throughput batch at t = 2^12
        dict(name="batch_4096", op="bootstrap", keys="paper", r="4", count=4096, general=False, plain=False, host=False),
        # users of different plaintext sizes in one host-memory call
        dict(name="mixed_811", op="bootstrap", keys="paper", r="1,2,4,8", count=811, general=False, plain=False, host=True),
        # a table too wide for one workgroup's components: t = 2^15
        dict(name="wide_table_100", op="bootstrap", keys="paper", r="16", count=100, general=False, plain=False, host=False),
        # a ternary secret, as Algorithm 1 is printed
        dict(name="ternary_300", op="bootstrap", keys="ternary", r="4", count=300, general=False, plain=False, host=False),
        # the same plaintext size by one ring of 4096 (the comparison scheme)
        dict(name="ring4096_700", op="bootstrap", keys="tfhe", r="1", count=700, general=False, plain=False, host=False),
        # the parameters of the paper's experiments: the identity on one ciphertext, two bootstraps
        dict(name="margin_one", op="bootstrap", keys="margin", r="128", count=1, general=True, plain=True, host=True),
        # the same for a batch at t = 2^9
        dict(name="margin_150", op="bootstrap", keys="margin", r="16", count=150, general=True, plain=False, host=False),
        # the steps alone, for programs that compose them: key switch, external product, ring product
        dict(name="keyswitch_1000", op="keyswitch", keys="paper", count=1000, host=False),
        dict(name="extprod_1000", op="external_product", keys="paper", count=1000, host=False),
        dict(name="ringmul_3000", op="negacyclic_mul", keys="paper", count=3000, host=False),
    ]


def _log_uniform(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["uniform", "uniform", "uniform", "mixed", "mixed", "ternary", "ring", "margin", "margin",
                       "keyswitch", "external_product", "negacyclic_mul"])
    host = rng.random() < 0.4
    if kind in ("keyswitch", "external_product", "negacyclic_mul"):
        return dict(op=kind, keys=rng.choice(["paper", "paper", "tfhe"]), count=_log_uniform(rng, 1, 4096), host=host)
    general = False
    if kind == "uniform":
        keys, r = "paper", rng.choice(["1", "2", "4", "4", "8", "16", "32"])
        top = 16384 // int(r)
    elif kind == "mixed":
        keys, r, top = "paper", rng.choice(["1,2,4,8", "1,4", "2,8", "4,16"]), 2048
    elif kind == "ternary":
        keys, r = "ternary", rng.choice(["1", "2", "4", "8"])
        top = 6000 // int(r)
    elif kind == "ring":
        keys, r, top = "tfhe", "1", 1500
    else:
        keys, r = "margin", rng.choice(["1", "2", "8", "16", "32", "64", "128"])
        general = rng.random() < 0.5
        top = max(1, (1200 if general else 2400) // int(r))
    count = _log_uniform(rng, 1, top)
    return dict(op="bootstrap", keys=keys, r=r, count=count, general=general, plain=count <= 4 and rng.random() < 0.5,
                host=host)


# ------------------------------------------------------------------ inputs

@lru_cache(maxsize=None)
def _draws(keys: str):
    return key_draws(KEY_SETS[keys], KEY_SEED)


@lru_cache(maxsize=None)
def _context(keys: str):
    ctx = binding.Context(KEY_SETS[keys], _draws(keys))
    ctx.device_init(0)
    return ctx


@lru_cache(maxsize=None)
def _table(keys: str, r: int, general: bool) -> int:
    t = plaintext_size(keys, r)
    ctx = _context(keys)
    if general:
        return ctx.table_create_general(t // 2, t // 2, r, np.arange(t // 2, dtype=np.uint32))  # the identity
    return ctx.table_create(t, t, r, negacyclic_table(t, t, 100 + r))


def _classes(case):
    return [int(x) for x in case["r"].split(",")]


def _ring_operands(case, seed):
    p = KEY_SETS[case["keys"]]
    rng = np.random.default_rng(seed)
    if case["op"] == "keyswitch":
        return [rng.integers(0, p.Q, size=(case["count"], p.N + 1), dtype=np.uint32)]
    if case["op"] == "external_product":
        return [rng.integers(0, p.Q, size=(case["count"], 2, p.N), dtype=np.uint32)]
    return [rng.integers(0, p.Q, size=(case["count"], p.N), dtype=np.uint32) for _ in range(2)]


def _place(a, host):
    return a if host else torch.from_numpy(a.view(np.int32)).cuda()


def prepare(case, seed):
    keys, count, host = case["keys"], case["count"], case["host"]
    p, ctx = KEY_SETS[keys], _context(keys)
    if case["op"] != "bootstrap":
        ins = [_place(a, host) for a in _ring_operands(case, seed)]
        shape = {"keyswitch": (count, p.n + 1), "external_product": (count, 2, p.N),
                 "negacyclic_mul": (count, p.N)}[case["op"]]
        out = np.empty(shape, np.uint32) if host else torch.empty(shape, dtype=torch.int32, device="cuda")
        return dict(case=case, ctx=ctx, ins=ins, out=out)
    classes = _classes(case)
    which = np.random.default_rng(seed).integers(0, len(classes), size=count)
    ids, cts = np.empty(count, np.int32), np.empty((count, p.n + 1), np.uint32)
    for k, r in enumerate(classes):
        sel = np.flatnonzero(which == k)
        q, t = 2 * p.N * r, plaintext_size(keys, r)
        ids[sel] = _table(keys, r, case["general"])
        if sel.size:
            e = enc_draws(p.n, q, sel.size, seed + 7919 * k)
            cts[sel] = ctx.encrypt(q, t, messages(t, sel.size, seed + 104729 * k), e["a"], e["e"])
    ins = _place(cts, host)
    return dict(case=case, ctx=ctx, ids=ids, ins=ins, out=np.empty_like(cts) if host else torch.empty_like(ins))


def run(state):
    case, ctx, out = state["case"], state["ctx"], state["out"]
    if case["op"] == "bootstrap":
        return ctx.bootstrap(state["ids"], state["ins"], plain=case["plain"], out=out)
    if case["op"] == "keyswitch":
        return ctx.keyswitch(state["ins"][0], out=out)
    if case["op"] == "external_product":
        return ctx.external_product(0, state["ins"][0], out=out)
    return ctx.negacyclic_mul(state["ins"][0], state["ins"][1], out=out)


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes: inputs, keys and outputs once each.  Operations: a butterfly is a product and
    two additions, a key product and its accumulation two operations, a key-switch row word one."""
    p = KEY_SETS[case["keys"]]
    N, n, l, count = p.N, p.n, p.l, case["count"]
    ntt = 3 * (N // 2) * (N.bit_length() - 1)
    primes, K = (2 if p.Q2 else 1), p.keys_per_coord
    product = primes * (K * (2 * l * ntt + 2 * 2 * l * N * 2) + 2 * ntt)  # one step of one component
    bsk, ksk = K * 2 * l * 2 * N * 4 * primes, N * p.l_ks * p.B_ks * (n + 1) * 4
    switch = N * p.l_ks * (n + 1)
    if case["op"] == "keyswitch":
        return {"bytes": count * (N + n + 2) * 4 + min(ksk, count * switch * 4), "flops": count * switch}
    if case["op"] == "external_product":
        return {"bytes": count * 4 * N * 4 + bsk // K, "flops": count * product // K}
    if case["op"] == "negacyclic_mul":
        return {"bytes": count * 3 * N * 4, "flops": count * (3 * ntt + N)}
    classes = _classes(case)
    comps = count * sum(classes) / len(classes)
    runs = 2 if case["general"] else 1
    return {"bytes": runs * (2 * count * (n + 1) * 4 + n * bsk + min(ksk, count * switch * 4)
                             + sum(classes) * primes * N * 4),
            "flops": int(runs * (comps * n * product + count * switch))}


# ------------------------------------------------------------------ the same results in 64 bits

def _negacyclic(a, b, Q):
    """a b mod (x^N + 1, Q) over the last axis: 16-bit limbs through complex FFTs of 64-bit
    floats (every limb product below 2^45, so the rounding is exact)."""
    N = a.shape[-1]
    twist = np.exp(1j * np.pi * np.arange(N) / N)

    def limbs(x):
        return [np.fft.fft(part.astype(np.float64) * twist) for part in (x & 0xFFFF, x >> 16)]

    def back(f):
        return np.rint((np.fft.ifft(f) / twist).real).astype(np.int64) % Q

    (a0, a1), (b0, b1) = limbs(a), limbs(b)
    mid = back(a0 * b1) + back(a1 * b0)
    return (back(a0 * b0) + (mid % Q) * 65536 + (back(a1 * b1) * 65536 % Q) * 65536) % Q


def _digits(x, p):
    """Signed gadget digits, low to high, of residues x: the nearest multiple of 2^sg in base 2^log2_B."""
    bits = p.Q.bit_length()
    sg, B = max(0, bits - p.l * p.log2_B), 1 << p.log2_B
    y = np.where(x > (p.Q - 1) // 2, x - p.Q, x)
    y = (y + (1 << sg >> 1)) >> sg
    out = []
    for u in range(p.l):
        d = y if u + 1 == p.l else (y + B // 2) % B - B // 2
        out.append(d)
        y = (y - d) >> p.log2_B
    return out, sg


def _exact_external_product(case, seed):
    p, d = KEY_SETS[case["keys"]], _draws(case["keys"])
    x = _ring_operands(case, seed)[0].astype(np.int64)
    z = d["z"].astype(np.int64)
    m = max(int(d["s"][0]), 0)
    out = np.zeros(x.shape, np.int64)
    for part, first in ((1, 0), (0, p.l)):  # digits of b meet rows u, digits of a rows l + u
        digits, sg = _digits(x[:, part], p)
        for u in range(p.l):
            a = d["bsk_a"][0, first + u].astype(np.int64)
            b = (_negacyclic(a, z, p.Q) + d["bsk_e"][0, first + u]) % p.Q
            (b if first == 0 else a)[0] += m * (1 << (sg + u * p.log2_B))
            for o, row in ((0, a % p.Q), (1, b % p.Q)):
                out[:, o] += _negacyclic(digits[u] % p.Q, row, p.Q)
    return (out % p.Q).astype(np.uint32)


def _exact_keyswitch(case, seed):
    p, d = KEY_SETS[case["keys"]], _draws(case["keys"])
    lwe = _ring_operands(case, seed)[0].astype(np.int64)
    rows = p.l_ks * p.B_ks
    s = d["s"].astype(np.float64)
    v = np.arange(p.B_ks)
    total = np.zeros((lwe.shape[0], p.n + 1))
    for i in range(p.N):
        key = np.empty((rows, p.n + 1))
        key[:, :p.n] = d["ksk_a"][i].reshape(rows, p.n)
        plain = np.concatenate([v * int(d["z"][i]) * (p.B_ks ** j % p.Q) % p.Q for j in range(p.l_ks)])
        key[:, p.n] = (key[:, :p.n] @ s + d["ksk_e"][i].reshape(rows) + plain) % p.Q
        pick = np.zeros((lwe.shape[0], rows))
        for j in range(p.l_ks):
            pick[np.arange(lwe.shape[0]), j * p.B_ks + ((lwe[:, i] >> (j * p.log2_Bks)) & (p.B_ks - 1))] = 1
        total += pick @ key  # sums of l_ks N residues: below 2^53, exact
    out = -total.astype(np.int64)
    out[:, p.n] += lwe[:, p.N]
    return (out % p.Q).astype(np.uint32)


def exact(case, seed):
    """The steps alone from the key draws; None for whole bootstraps (minutes in plain
    numpy) and for the key switches and products that take too long there."""
    p, op = KEY_SETS[case["keys"]], case["op"]
    if op == "negacyclic_mul":
        a, b = _ring_operands(case, seed)
        want = _negacyclic(a.astype(np.int64), b.astype(np.int64), p.Q).astype(np.uint32)
    elif op == "external_product" and case["count"] * p.N <= 1 << 20:
        want = _exact_external_product(case, seed)
    elif op == "keyswitch" and case["count"] * p.N <= 1 << 20:
        want = _exact_keyswitch(case, seed)
    else:
        return None
    return want if case["host"] else want.view(np.int32)
