// Device code shared by the blind-rotation kernels: the modulus switch of a coordinate,
// the rows of Phi, a wave's task in scalar registers and the order of work items.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>

#include "kernels.hpp"

namespace mm {
namespace dev {

// a' = round(x M / q) (Sec. 2 item (9)), ties upward.
__device__ __forceinline__ uint32_t wide_modswitch(uint32_t x, uint32_t q, uint32_t M)
{
    return (uint32_t)(((2ull * x * M + q) / (2ull * q)) % M);
}

// Row j of Phi(c) for c = a r + b (eq. ex1:BPc): source component (j - b) mod r
// and monomial x^(a + [j < b]), returned as a shift e in [0, N) and a sign.
struct WideRow {
    uint32_t src, e;
    bool neg;
};

__device__ __forceinline__ WideRow wide_row(uint32_t c, uint32_t r, uint32_t j, uint32_t N)
{
    const uint32_t a = c / r, b = c - a * r;
    WideRow w;
    w.src = j >= b ? j - b : j + r - b;
    uint32_t e = (a + (j < b ? 1u : 0u)) % (2 * N);
    w.neg = e >= N;
    w.e = w.neg ? e - N : e;
    return w;
}

// Coefficient idx of x^e p (negacyclic, e < N): p[idx - e], negated when the
// index wraps; `neg` folds in a further x^N = -1.
__device__ __forceinline__ uint32_t wide_rot_load(const uint32_t *p, uint32_t idx, const WideRow &w, uint32_t N,
                                                  uint32_t Q)
{
    const uint32_t v = p[(idx - w.e) & (N - 1)];
    const bool flip = (idx < w.e) != w.neg;
    return (flip && v) ? Q - v : v;
}

// Work item of workgroup b of a grid of g: the hardware deals workgroups to the eight
// XCDs in turn (b mod 8), each with its own L2; this mapping gives each XCD a contiguous
// eighth of the items (the rest, g mod 8, in order), so the components of one
// ciphertext -- which read each other's accumulators through the rotation -- share an L2.
__device__ __forceinline__ uint32_t xcd_item(uint32_t b, uint32_t g)
{
    const uint32_t full = g / 8 * 8;
    return b < full ? (b % 8) * (full / 8) + b / 8 : b;
}

__device__ __forceinline__ uint32_t modswitch_dev(uint32_t x, uint32_t q_from, uint32_t q_to)
{
    if (q_from == q_to) return x;
    const uint64_t num = 2ull * (uint64_t)x * q_to + q_from;
    return (uint32_t)((num / (2ull * q_from)) % q_to);
}

// Row j of Phi(c), c = a r + b: source component (j - b) mod r and monomial
// exponent a + [j < b] (eq. ex1:BPc).
__device__ __forceinline__ void phi_row(uint32_t c, uint32_t r, uint32_t j, uint32_t &src, uint32_t &e)
{
    const uint32_t a = c / r, b = c - a * r;
    src = (j + r - b) % r;
    e = a + (j < b ? 1u : 0u);
}

// A wave's task, every field moved to scalar registers (the same for all lanes),
// so that the step index, key and ciphertext addresses derived from it stay
// scalar and the per-lane part of each address is one 32-bit offset.
__device__ __forceinline__ WaveTask uniform_task(const WaveTask &t)
{
    WaveTask u;
    u.ct = __builtin_amdgcn_readfirstlane(t.ct);
    u.comp = __builtin_amdgcn_readfirstlane(t.comp);
    u.r = __builtin_amdgcn_readfirstlane(t.r);
    u.tv_off = __builtin_amdgcn_readfirstlane(t.tv_off);
    u.q_in = __builtin_amdgcn_readfirstlane(t.q_in);
    u.i0 = __builtin_amdgcn_readfirstlane(t.i0);
    u.flags = __builtin_amdgcn_readfirstlane(t.flags);
    u.steps = __builtin_amdgcn_readfirstlane(t.steps);
    u.acc_off = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(t.acc_off >> 32)) << 32) |
                __builtin_amdgcn_readfirstlane((uint32_t)t.acc_off);
    return u;
}

}  // namespace dev
}  // namespace mm
