// The CMux step, the external product and the ring product on the matrix cores: one prime
// below 2^31 at N = 1024 with digits of at most 7 bits, two primes at N = 2048 with digits of
// at most 15.
//
// The negacyclic NTT of N = 32 x 32 points in two 32-point stages,
//   X[k1 + 32 k2] = sum_i2 w^(i2 k2) psi^(i2 (2 k1 + 1)) sum_i1 x[32 i1 + i2] psi^(32 i1 (2 k1 + 1)),
// w = psi^64, is two products with constant 32 x 32 matrices and one product by
// twiddles in between.  Both matrix products run as v_mfma_i32_32x32x32_i8 on
// signed bytes: the matrices are held in four balanced byte limbs, the digits of
// the gadget are bytes already (|d| <= 64), and a 32-bit residue enters a product
// as its own four balanced bytes along the contraction, row (i, m) of the
// constant being 2^(8m) times row i.  The four limb sums of an output are below
// 2^22 and recombine to lo + 2^16 hi in two shift-adds; a 64-bit multiply-add and
// a Montgomery reduction give the next residue.  Every step is exact, so results
// equal those of the butterfly network bit for bit.
//
// Layout: lane (c = lane % 32, h = lane / 32) of a wave, register v = 4 q + s holds
// row 8 q + 4 h + s of column c -- the accumulator layout of the instruction.  A
// residue's four bytes are one register, and registers 4 q .. 4 q + 3 of the two
// lane halves are exactly the 32-byte operand of a contraction over rows
// 8 q .. 8 q + 7: the output of one product is the operand of the next, with no
// exchange between lanes at all.  The inverse runs the same way from the other
// side (the values as the left operand, so that its output has k1 in the rows).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "rotation_common.hpp"
#include "wrap64.hpp"

namespace mm {
namespace dev {

typedef int32_t v4i __attribute__((ext_vector_type(4)));
typedef int32_t v16i __attribute__((ext_vector_type(16)));

constexpr int MXN = 1024;
constexpr uint32_t BAL = 0x80808080u;  // x + BAL, then xor BAL: the four balanced bytes of x

struct ModS {
    int32_t Q;    // odd modulus < 2^31
    uint32_t qn;  // -Q^-1 mod 2^32
};

// o = (t 2^-32 mod Q) + the high word of whatever was added to t's high word beforehand,
// in wrapping 32 bits; without such a bias a signed representative of magnitude at most
// |t| / 2^32 + Q / 2.  Four at a time: the empty asm keeps every sum in one piece (its
// reassociation into the reduction costs an addition) and the four chains abreast.
__device__ __forceinline__ void redc4(int64_t (&t)[4], const ModS &m, int32_t (&o)[4])
{
    __asm__("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]));
    int32_t q[4];
#pragma unroll
    for (int s = 0; s < 4; s++) q[s] = (int32_t)((uint32_t)t[s] * m.qn);
    __asm__("" : "+v"(q[0]), "+v"(q[1]), "+v"(q[2]), "+v"(q[3]));
#pragma unroll
    for (int s = 0; s < 4; s++) o[s] = (int32_t)(mad_wrap(q[s], m.Q, t[s]) >> 32);
}

__device__ __forceinline__ v16i mfma(v4i a, v4i b, v16i c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0); }

// The constant block (mx_tables in device.cpp), operands of 64 lanes x 16 bytes: the first
// stage's four limbs, the second stage's [contraction block][limb], the forward twiddles
// [block][w, 2^16 w], the last inverse stage's row factors [block][lane half][f, 2^16 f]
// -- these in LDS -- and the inverse twiddles, read once per step from memory.  The inverse
// stages use the second stage's matrix at the negated column (w^(-a b) = w^(a (32 - b))).
enum { MX_FA = 0, MX_FB = 4, MX_TWF = 20, MX_FIN = 28 };
constexpr int MX_VECS = MX_FIN * 64 + 16;
constexpr int MX_FR = MX_VECS + 8 * 64;  // the first stage for residues, [contraction block][limb] (k_mx_ring)
static_assert((MX_FR + 16 * 64) * 4 == (int)MX_CONST_WORDS, "constant block size");

// A workgroup's copy of ops operands into LDS, DEPTH requests per thread in flight.
template <int DEPTH = 4, class Src>
__device__ __forceinline__ void mx_copy(int ops, Src src, v4i *dst)
{
    for (int t0 = threadIdx.x; t0 < ops; t0 += DEPTH * (int)blockDim.x) {
        v4i x[DEPTH];
#pragma unroll
        for (int k = 0; k < DEPTH; k++) x[k] = src(min(t0 + k * (int)blockDim.x, ops - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < DEPTH; k++) dst[min(t0 + k * (int)blockDim.x, ops - 1)] = x[k];
    }
}

// Position of register v of a lane: row 8 (v / 4) + 4 half + v % 4, 32 words per row.
__device__ __forceinline__ int mx_off(int v) { return 256 * (v / 4) + 32 * (v % 4); }

// Two limb sums joined (upper: limbs 2 and 3, or limb 2 alone with NL = 3).
template <int NL>
__device__ __forceinline__ void mx_join(bool upper, const v16i &a, const v16i &b, int32_t (&o)[16])
{
#pragma unroll
    for (int v = 0; v < 16; v++) o[v] = upper && NL == 3 ? a[v] : a[v] + (int32_t)((uint32_t)b[v] << 8);
}

// One 32-point stage on a residue polynomial given as bytes: the four limb sums of each
// output joined to lo + 2^16 hi, two limbs at a time.  LEFT: the constant is the left
// operand.  work(t), t = 0 .. 7, is vector arithmetic of another polynomial placed after
// every second instruction: alone, a wave's matrix instructions would leave the vector
// ALU idle and its arithmetic the matrix unit (40 matrix instructions and 480 others of
// this mix take 3.7k clocks per wave one after the other, 3.2k interleaved, at two waves
// per SIMD).
// NL = 3: constants of at most 23 bits have three limbs, hi is the third alone (operands
// [contraction block][NL]).
template <bool LEFT, int NL = 4, class Work>
__device__ __forceinline__ void mx_stage(const v4i *fb, const v4i (&z)[4], int lane, int32_t (&lo)[16],
                                         int32_t (&hi)[16], Work work)
{
    v4i k[2] = {fb[lane], fb[64 + lane]};
    v16i c[2];
#pragma unroll
    for (int t = 0; t < 8; t++) {
        const int q = t & 3, nj = t < 4 ? 2 : NL - 2;
        if (q == 0) c[0] = c[1] = v16i{};
#pragma unroll
        for (int j = 0; j < nj; j++) c[j] = LEFT ? mfma(k[j], z[q], c[j]) : mfma(z[q], k[j], c[j]);
        if (t < 7) {
#pragma unroll
            for (int j = 0; j < (t < 3 ? 2 : NL - 2); j++)
                k[j] = fb[(NL * ((t + 1) & 3) + 2 * ((t + 1) >> 2) + j) * 64 + lane];
        }
        work(t);
        if (q == 3) mx_join<NL>(t == 7, c[0], c[1], t == 7 ? hi : lo);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Half a step (t = 2 q + half) of: lo + 2^16 hi times the twiddles (w, 2^16 w, in
// Montgomery form), as balanced bytes z[q].
__device__ __forceinline__ void mx_twist(int t, const int32_t (&lo)[16], const int32_t (&hi)[16], const v4i *tw, int pitch,
                                         const MxArgs &X, const ModS &m, int64_t (&s4)[4], v4i (&z)[4])
{
    const int q = t >> 1;
    if (!(t & 1)) {
        const v4i w = tw[2 * q * pitch], w16 = tw[(2 * q + 1) * pitch];
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = mad_wrap(hi[4 * q + s], w16[s], X.bal64);
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = mad_wrap(lo[4 * q + s], w[s], s4[s]);
    } else {
        int32_t o[4];
        redc4(s4, m, o);
#pragma unroll
        for (int s = 0; s < 4; s++) z[q][s] = o[s] ^ (int32_t)BAL;
    }
}

// Half a step of: the NTT values lo + 2^16 hi times both parts' key words, added to acc.
__device__ __forceinline__ void mx_mac(int t, const int32_t (&lo)[16], const int32_t (&hi)[16], const v4i (&k)[2][4],
                                       const MxArgs &X, const ModS &m, int32_t (&r4)[4], int64_t (&acc)[2][16])
{
    const int q = t >> 1;
    if (!(t & 1)) {
        int64_t s4[4];
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = (int64_t)hi[4 * q + s] * X.two16 + lo[4 * q + s];
        redc4(s4, m, r4);
    } else {
#pragma unroll
        for (int o = 0; o < 2; o++)
#pragma unroll
            for (int s = 0; s < 4; s++) acc[o][4 * q + s] += (int64_t)r4[s] * k[o][q][s];
    }
}

// Digit u of the fields y of P parts as signed bytes ([u][part]), the first stage's operand,
// into the wave's LDS (each lane reads back only its own); with one part a zero polynomial
// behind an odd number of digits.
template <int P>
__device__ __forceinline__ void mx_digits(const uint32_t (&y)[P][16], uint32_t l, uint32_t log2B, const MxArgs &X,
                                          int lane, v4i *dig)
{
#pragma unroll
    for (uint32_t u = 0; u < MX_MAX_L; u++) {
        if (u >= l) break;
        const uint32_t sh = u * log2B, wd = log2B + (u + 1 == l ? 1u : 0u);
#pragma unroll
        for (int part = 0; part < P; part++) {
            v4i d;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                uint32_t p = 0;
#pragma unroll
                for (int s = 0; s < 4; s++) p |= __builtin_amdgcn_ubfe(y[part][4 * q + s], sh, wd) << (8 * s);
                d[q] = (int32_t)((p + X.bias) ^ BAL);
            }
            dig[(P * u + part) * 64 + lane] = d;
        }
    }
    if (P == 1 && (l & 1)) dig[l * 64 + lane] = v4i{};
}

// acc += two digit polynomials (operands x) times their key rows kr.
__device__ __forceinline__ void mx_pair(const v4i (&x)[2], const v4i *const (&kr)[2], const v4i *cst, int lane,
                                        const MxArgs &X, const ModS &m, int64_t (&acc)[2][16])
{
    int32_t lo[2][16], hi[2][16];
    v4i z[2][4], k[2][2][4];
    int64_t s4[4];
    int32_t r4[4];
    auto request = [&](int p) {
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int o = 0; o < 2; o++) k[p][o][q] = kr[p][(4 * o + q) * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int p = 0; p < 2; p++) {
        v16i c[4];
#pragma unroll
        for (int j = 0; j < 4; j++) c[j] = mfma(x[p], cst[(MX_FA + j) * 64 + lane], v16i{});
        if (p == 1) {
#pragma unroll
            for (int t = 0; t < 8; t++) mx_twist(t, lo[0], hi[0], cst + MX_TWF * 64 + lane, 64, X, m, s4, z[0]);
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
            lo[p][v] = c[0][v] + (int32_t)((uint32_t)c[1][v] << 8);
            hi[p][v] = c[2][v] + (int32_t)((uint32_t)c[3][v] << 8);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    request(0);
    mx_stage<true>(cst + MX_FB * 64, z[0], lane, lo[0], hi[0],
                   [&](int t) { mx_twist(t, lo[1], hi[1], cst + MX_TWF * 64 + lane, 64, X, m, s4, z[1]); });
    request(1);
    mx_stage<true>(cst + MX_FB * 64, z[1], lane, lo[1], hi[1], [&](int t) { mx_mac(t, lo[0], hi[0], k[0], X, m, r4, acc); });
#pragma unroll
    for (int t = 0; t < 8; t++) mx_mac(t, lo[1], hi[1], k[1], X, m, r4, acc);
}

// Row of the key block K as operand words.
__device__ __forceinline__ const v4i *mx_row(const int32_t *K, uint32_t row)
{
    return reinterpret_cast<const v4i *>(K + (size_t)row * 2 * MXN);
}

// acc += the digit polynomials of both parts ([u][part]) times their key rows: digits of a
// (part 0) meet rows l + u, digits of b rows u (eq. def:gsw).
__device__ __forceinline__ void mx_products(const v4i *dig, const v4i *cst, const int32_t *K, uint32_t l, int lane,
                                            const MxArgs &X, const ModS &m, int64_t (&acc)[2][16])
{
    for (uint32_t u = 0; u < l; u++) {
        __asm__ volatile("" ::: "memory");  // constants and key words are read where they are used
        const v4i x[2] = {dig[2 * u * 64 + lane], dig[(2 * u + 1) * 64 + lane]};
        const v4i *const kr[2] = {mx_row(K, l + u), mx_row(K, u)};
        mx_pair(x, kr, cst, lane, X, m, acc);
    }
}

// The same for one part's digits ([u], a zero polynomial behind an odd number), by pairs of u.
__device__ __forceinline__ void mx_products_part(const v4i *dig, int part, const v4i *cst, const int32_t *K, uint32_t l,
                                                 int lane, const MxArgs &X, const ModS &m, int64_t (&acc)[2][16])
{
    const uint32_t first = part ? 0 : l;
    for (uint32_t u = 0; u < l; u += 2) {
        __asm__ volatile("" ::: "memory");
        const v4i x[2] = {dig[u * 64 + lane], dig[(u + 1) * 64 + lane]};
        const v4i *const kr[2] = {mx_row(K, first + u), mx_row(K, first + min(u + 1, l - 1))};
        mx_pair(x, kr, cst, lane, X, m, acc);
    }
}

// Registers 4 q .. 4 q + 3 of one part's sums as balanced bytes of their residues x 2^-32:
// 2^32 h + l -> h (2^32 mod Q) + l, which one reduction brings below 2^31; BAL as its bias.
__device__ __forceinline__ void mx_cut(int q, const int64_t (&acc)[16], const MxArgs &X, const ModS &m, int64_t (&s4)[4],
                                       v4i (&z)[4])
{
    int32_t o[4];
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const uint64_t low = (uint32_t)acc[4 * q + s] | ((uint64_t)BAL << 32);
        s4[s] = mad_wrap((int32_t)(acc[4 * q + s] >> 32), X.two32, (int64_t)low);
    }
    redc4(s4, m, o);
#pragma unroll
    for (int s = 0; s < 4; s++) z[q][s] = o[s] ^ (int32_t)BAL;
}

// The sums back to coefficients: out(part, v, x) with x in [0, Q).
template <class Out>
__device__ __forceinline__ void mx_inverse(const int64_t (&acc)[2][16], const v4i *cst, int lane, const MxArgs &X,
                                           const ModS &m, Out out)
{
    __asm__ volatile("" ::: "memory");
    const int neg = ((32 - lane) & 31) | (lane & 32);
    int32_t lo[2][16], hi[2][16];
    v4i z[2][4], tw[8];
    int64_t s4[4];
    // the inverse twiddles, requested before the first stage
#pragma unroll
    for (int j = 0; j < 8; j++) tw[j] = reinterpret_cast<const v4i *>(X.cst)[MX_VECS + j * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
    auto cut = [&](int p, int q) { mx_cut(q, acc[p], X, m, s4, z[p]); };
    auto twist = [&](int p, int t) { mx_twist(t, lo[p], hi[p], tw, 1, X, m, s4, z[p]); };
    auto last = [&](int p, int q) {
        const v4i f = cst[MX_FIN * 64 + 4 * q + 2 * (lane >> 5)], f16 = cst[MX_FIN * 64 + 4 * q + 2 * (lane >> 5) + 1];
        int32_t o[4];
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = (int64_t)lo[p][4 * q + s] * f[s] + (int64_t)hi[p][4 * q + s] * f16[s];
        redc4(s4, m, o);
#pragma unroll
        for (int s = 0; s < 4; s++) out(p, 4 * q + s, min((uint32_t)o[s], (uint32_t)o[s] + (uint32_t)m.Q));  // o in (-Q, Q)
    };
#pragma unroll
    for (int q = 0; q < 4; q++) cut(0, q);
    mx_stage<false>(cst + MX_FB * 64, z[0], neg, lo[0], hi[0], [&](int t) { if (t & 1) cut(1, t >> 1); });
    mx_stage<false>(cst + MX_FB * 64, z[1], neg, lo[1], hi[1], [&](int t) { twist(0, t); });
    mx_stage<true>(cst + MX_FB * 64, z[0], neg, lo[0], hi[0], [&](int t) { twist(1, t); });
    mx_stage<true>(cst + MX_FB * 64, z[1], neg, lo[1], hi[1], [&](int t) { if (t & 1) last(0, t >> 1); });
#pragma unroll
    for (int q = 0; q < 4; q++) last(1, q);
}

// The same for one part alone: out(v, x).
template <class Out>
__device__ __forceinline__ void mx_inverse_part(const int64_t (&acc)[16], const v4i *cst, int lane, const MxArgs &X,
                                                const ModS &m, Out out)
{
    __asm__ volatile("" ::: "memory");
    const int neg = ((32 - lane) & 31) | (lane & 32);
    int32_t lo[16], hi[16], o[4];
    v4i z[4], tw[8];
    int64_t s4[4];
#pragma unroll
    for (int j = 0; j < 8; j++) tw[j] = reinterpret_cast<const v4i *>(X.cst)[MX_VECS + j * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; q++) mx_cut(q, acc, X, m, s4, z);
    mx_stage<false>(cst + MX_FB * 64, z, neg, lo, hi, [](int) {});
#pragma unroll
    for (int t = 0; t < 8; t++) mx_twist(t, lo, hi, tw, 1, X, m, s4, z);
    mx_stage<true>(cst + MX_FB * 64, z, neg, lo, hi, [](int) {});
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const v4i f = cst[MX_FIN * 64 + 4 * q + 2 * (lane >> 5)], f16 = cst[MX_FIN * 64 + 4 * q + 2 * (lane >> 5) + 1];
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = (int64_t)lo[4 * q + s] * f[s] + (int64_t)hi[4 * q + s] * f16[s];
        redc4(s4, m, o);
#pragma unroll
        for (int s = 0; s < 4; s++) out(4 * q + s, min((uint32_t)o[s], (uint32_t)o[s] + (uint32_t)m.Q));
    }
}

// Sums of one key's products, folded so that another key's fit on top below 2^63.
__device__ __forceinline__ void mx_fold(int64_t (&acc)[2][16], const MxArgs &X)
{
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int v = 0; v < 16; v++)
            acc[p][v] = (int64_t)(int32_t)(acc[p][v] >> 32) * X.two32 + (int64_t)(uint64_t)(uint32_t)acc[p][v];
}

// Two waves per component: the sums of the other part to its wave, through LDS, ...
__device__ __forceinline__ void mx_give(const int64_t (&acc)[2][16], int part, int lane, v4i *sums)
{
#pragma unroll
    for (int v = 0; v < 8; v++) {
        const int64_t t0 = part ? acc[0][2 * v] : acc[1][2 * v];
        const int64_t t1 = part ? acc[0][2 * v + 1] : acc[1][2 * v + 1];
        sums[v * 64 + lane] = v4i{(int32_t)t0, (int32_t)(t0 >> 32), (int32_t)t1, (int32_t)(t1 >> 32)};
    }
}

// ... and, a barrier later, this part's sums of both waves.
__device__ __forceinline__ void mx_take(const int64_t (&acc)[2][16], int part, int lane, const v4i *sums,
                                        int64_t (&mine)[16])
{
#pragma unroll
    for (int v = 0; v < 8; v++) {
        const v4i t = sums[v * 64 + lane];
        const int64_t t0 = (int64_t)((uint64_t)(uint32_t)t[1] << 32 | (uint32_t)t[0]);
        const int64_t t1 = (int64_t)((uint64_t)(uint32_t)t[3] << 32 | (uint32_t)t[2]);
        mine[2 * v] = (part ? acc[1][2 * v] : acc[0][2 * v]) + t0;
        mine[2 * v + 1] = (part ? acc[1][2 * v + 1] : acc[0][2 * v + 1]) + t1;
    }
}

// The digit fields of D = src - own, or Q - src - own where the rotation negates src (flip
// all ones): one min brings it to [0, Q), another moves the values above (Q - 1) / 2 below 0
// (offset by (Q - 1) / 2), and centring, rounding and digit offset are one constant before
// the shift (their sum is never negative).
__device__ __forceinline__ uint32_t mx_field(uint32_t src, uint32_t own, uint32_t flip, uint32_t fq, uint32_t Q,
                                             const MxArgs &X, uint32_t sg)
{
    uint32_t t = (src ^ flip) + (fq - own);  // in (-Q, Q]
    t = min(t, t + Q) + (Q - 1) / 2;         // in [0, 2 Q)
    t = min(t, t - Q);
    return (t + X.field) >> sg;
}

// ------------------------------------------------------------------ the fused blind rotation

// All n CMux steps of up to eight ring components per workgroup, W = 1 wave per component
// (the groups and tasks of k_blind_rotate): the accumulators stay in LDS, one buffer,
// two workgroup barriers per step (every rotation has read; every component is written).
//
// Bound by vector issue: a component's step is 3,440 vector and 224 matrix instructions
// (69 % of the four-clock issue slots; the matrix unit is busy 34 % of the time and each of
// its instructions holds vector issue for about 12 clocks), at the 2.0 GHz the device runs
// under this load.  Two waves per SIMD: 256 registers hold the 64-bit sums (64), two
// polynomials' values and the key words in flight; LDS holds the constants (29 KB), the
// digits (64 KB) and the accumulators (64 KB) of eight waves.  Measured for 16,384 components,
// 630 steps: 102 ms, against 183 for k_wide_step<1024, 1, 1, 4> and 204 for k_blind_rotate;
// one workgroup alone 7.4 ms with one wave per SIMD, 12.8 with two.
//
// W = 2: two waves per component, up to four components: wave p takes part p of the rotation,
// its digits' products onto both parts' sums, and part p of the inverse; the sums of the
// other part go to its wave through LDS before the second barrier.
template <int KEYS, int W>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_rotate(BrArgs A)
{
    constexpr int P = 2 / W;  // parts per wave
    __shared__ v4i cst[MX_VECS];
    __shared__ v4i digits[8][MX_MAX_L * P * 64];
    __shared__ uint32_t accs[8 / W][2 * MXN];
    __shared__ v4i sums[W == 2 ? 8 : 1][8 * 64];
    mx_copy(MX_VECS, [&](int t) { return reinterpret_cast<const v4i *>(A.mx.cst)[t]; }, cst);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = (lane & 31) + 128 * (lane >> 5);  // + mx_off(v): the coefficient of register v
    const int slot = wave / W, p0 = W == 2 ? wave & 1 : 0;
    uint32_t *const own = accs[slot] + p0 * MXN + base;
    v4i *const dig = digits[wave];
    const uint32_t Q = A.Q;
    const ModS m{(int32_t)Q, A.qn};
    for (int grp = blockIdx.x; grp < A.num_groups; grp += gridDim.x) {
        const WaveTask T = uniform_task(A.tasks[grp * 8 + wave]);
        const bool has = T.ct >= 0;
        const uint32_t r = has ? T.r : 1u, M = 2u * MXN * r;
        const uint32_t *ct = A.ct_in + (size_t)(has ? T.ct : 0) * A.ct_stride;
        // an opaque copy of the lane's position: the addresses of a group's ends stay out of the steps
        int pos = base;
        __asm__("" : "+v"(pos));
        uint32_t *const mine = accs[slot] + p0 * MXN + pos;
        // Phi(b') (0, V) or the stored state; each lane writes the words it alone reads back
        // as its own, and the step's first barrier makes them visible to the rotations
        if (has && (T.flags & TASK_INIT)) {
            uint32_t src, e;
            phi_row(__builtin_amdgcn_readfirstlane(modswitch_dev(ct[A.n], T.q_in, M)), r, T.comp, src, e);
            const uint32_t *V = A.tv + T.tv_off + (size_t)src * MXN;
#pragma unroll
            for (int p = 0; p < P; p++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    uint32_t x = 0;
                    if (p0 + p == 1) {
                        const uint32_t i2 = (pos + mx_off(v) + 2 * MXN - (e % (2 * MXN))) % (2 * MXN);
                        x = V[i2 & (MXN - 1)];
                        if (i2 >= (uint32_t)MXN) x = x ? Q - x : 0;
                    }
                    mine[p * MXN + mx_off(v)] = x;
                }
        } else if (has) {
            const uint32_t *S = A.acc_state + T.acc_off + (size_t)T.comp * 2 * MXN + p0 * MXN + pos;
#pragma unroll
            for (int p = 0; p < P; p++)
#pragma unroll
                for (int v = 0; v < 16; v++) mine[p * MXN + mx_off(v)] = S[p * MXN + mx_off(v)];
        }
        const uint32_t lim = T.steps ? min(T.steps, (uint32_t)A.steps) : (uint32_t)A.steps;
        for (int s = 0; s < A.steps; s++) {
            const uint32_t i = T.i0 + (uint32_t)s;
            const bool active = has && i < A.n && (uint32_t)s < lim;
            __syncthreads();  // every accumulator is written (and, at first, the constants)
            int64_t acc[2][16];
            if (active) {
                const uint32_t am = __builtin_amdgcn_readfirstlane(modswitch_dev(ct[i], T.q_in, M));
#pragma unroll
                for (int v = 0; v < 16; v++) acc[0][v] = acc[1][v] = 0;
#pragma unroll 1
                for (int key = 0; key < KEYS; key++) {
                    uint32_t src, e;
                    phi_row(key == 0 ? (M - am) % M : am, r, T.comp, src, e);
                    const uint32_t *sp = accs[slot - T.comp + src] + p0 * MXN;
                    const uint32_t rb = (uint32_t)base + 2 * MXN - (e % (2 * MXN));
                    uint32_t y[P][16];
#pragma unroll
                    for (int v = 0; v < 16; v++) {
                        const uint32_t i2 = rb + mx_off(v);
                        const uint32_t at = i2 & (MXN - 1);
                        const uint32_t flip = 0u - ((i2 >> 10) & 1u);
                        const uint32_t fq = flip & (Q + 1);
#pragma unroll
                        for (int p = 0; p < P; p++)
                            y[p][v] = mx_field(sp[p * MXN + at], own[p * MXN + mx_off(v)], flip, fq, Q, A.mx, A.sg);
                    }
                    mx_digits<P>(y, A.l, A.log2B, A.mx, lane, dig);
                    const int32_t *K = A.mx.bsk + ((size_t)i * KEYS + key) * (4u * A.l * MXN);
                    if constexpr (W == 1) mx_products(dig, cst, K, A.l, lane, A.mx, m, acc);
                    else mx_products_part(dig, p0, cst, K, A.l, lane, A.mx, m, acc);
                    if (KEYS == 2 && key == 0) mx_fold(acc, A.mx);
                }
                if constexpr (W == 2) {
                    mx_give(acc, p0, lane, sums[wave]);
                }
            }
            __syncthreads();  // every rotation of the step has read the accumulators
            if (active) {
                auto store = [&](int p, int v, uint32_t x) {
                    uint32_t *o = own + p * MXN + mx_off(v);
                    *o = add_q(*o, x, Q);
                };
                if constexpr (W == 1) {
                    mx_inverse(acc, cst, lane, A.mx, m, store);
                } else {
                    int64_t mysum[16];
                    mx_take(acc, p0, lane, sums[wave ^ 1], mysum);
                    mx_inverse_part(mysum, cst, lane, A.mx, m, [&](int v, uint32_t x) { store(0, v, x); });
                }
            }
        }
        if (has) {
            if (T.flags & TASK_STORE) {
                uint32_t *S = A.acc_state + T.acc_off + (size_t)T.comp * 2 * MXN + p0 * MXN + pos;
#pragma unroll
                for (int p = 0; p < P; p++)
#pragma unroll
                    for (int v = 0; v < 16; v++) S[p * MXN + mx_off(v)] = mine[p * MXN + mx_off(v)];
            }
            if ((T.flags & TASK_EXTRACT) && T.comp == 0 && T.i0 + lim >= A.n) {
                // (A_0, -A_{N-1}, ..., -A_1; B_0) (eq. equ-sam-extr)
                uint32_t *o = A.ext_out + (size_t)T.ct * (MXN + 1);
                if (p0 == 0) {
#pragma unroll
                    for (int v = 0; v < 16; v++) {
                        const uint32_t idx = pos + mx_off(v), x = mine[mx_off(v)];
                        o[(MXN - idx) & (MXN - 1)] = idx ? (x ? Q - x : 0) : x;
                    }
                }
                if (p0 + P == 2 && lane == 0) o[MXN] = mine[(1 - p0) * MXN];
            }
        }
        __syncthreads();  // the next group's accumulators take this one's place
    }
}

// ------------------------------------------------------------------ external products

// g^{-1}(in) x one key of `count` pairs [count][2][N] -> out: the step without a rotation, W
// waves per pair as in k_mx_rotate, four pairs per workgroup, the key words shared by all.
//
// Bound by the chain of one wave (as a step of k_mx_rotate) up to one workgroup per compute
// unit, by vector issue beyond.  Measured against k_external_product<1024>, us per call in a row,
// pairs in the last-level cache / streamed through 1.2 GB: 1 pair 11.7 / 11.5 against 24.1, 1000 13.1 /
// 15.8 (1.25 / 1.04 TB/s of pairs read and written) against 28.2 / 29.8, 4096 46.0 / 48.4 against 83.4 /
// 84.5, 20,000 225 against 387.  With one wave per pair two workgroups share a compute unit and
// one's loads run under the other's arithmetic (workgroups of eight pairs: 9 % longer at 4096).
template <int W>
__global__ __launch_bounds__(256 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_product(
    MxArgs X, const uint32_t *in, uint32_t *out, size_t count, uint32_t key, uint32_t Q, uint32_t qn, uint32_t log2B,
    uint32_t l, uint32_t sg)
{
    constexpr int P = 2 / W;
    __shared__ v4i cst[MX_VECS];
    __shared__ v4i digits[4 * W][MX_MAX_L * P * 64];
    __shared__ v4i sums[W == 2 ? 8 : 1][8 * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = (lane & 31) + 128 * (lane >> 5), p0 = W == 2 ? wave & 1 : 0;
    const size_t item = (size_t)blockIdx.x * 4 + wave / W;
    const bool has = item < count;
    v4i *const dig = digits[wave];
    const ModS m{(int32_t)Q, qn};
    const size_t at = (has ? item : 0) * 2 * MXN + p0 * MXN + base;
    uint32_t x[P][16];
#pragma unroll
    for (int p = 0; p < P; p++)
#pragma unroll
        for (int v = 0; v < 16; v++) x[p][v] = in[at + p * MXN + mx_off(v)];
    mx_copy(MX_VECS, [&](int t) { return reinterpret_cast<const v4i *>(X.cst)[t]; }, cst);
    __syncthreads();
    int64_t acc[2][16];
    if (has) {
#pragma unroll
        for (int p = 0; p < P; p++)
#pragma unroll
            for (int v = 0; v < 16; v++) x[p][v] = mx_field(x[p][v], 0, 0, 0, Q, X, sg);
        mx_digits<P>(x, l, log2B, X, lane, dig);
#pragma unroll
        for (int v = 0; v < 16; v++) acc[0][v] = acc[1][v] = 0;
        const int32_t *K = X.bsk + (size_t)key * (4u * l * MXN);
        if constexpr (W == 1) mx_products(dig, cst, K, l, lane, X, m, acc);
        else mx_products_part(dig, p0, cst, K, l, lane, X, m, acc);
    }
    auto store = [&](int p, int v, uint32_t c) { out[at + p * MXN + mx_off(v)] = c; };
    if constexpr (W == 1) {
        if (has) mx_inverse(acc, cst, lane, X, m, store);
    } else {
        if (has) mx_give(acc, p0, lane, sums[wave]);
        __syncthreads();
        if (has) {
            int64_t mysum[16];
            mx_take(acc, p0, lane, sums[wave ^ 1], mysum);
            mx_inverse_part(mysum, cst, lane, X, m, [&](int v, uint32_t c) { store(0, v, c); });
        }
    }
}

// ------------------------------------------------------------------ ring products

// a b of `count` pairs of polynomials [count][N], one wave per product.  The operands are
// residues, not digits, so the first stage too contracts over their balanced bytes.
//
// Bound by vector issue beside the matrix instructions (970 and 96 per product).  One workgroup
// per compute unit of up to three waves per SIMD (165 registers); the constants (41 KB) are read
// once, a wave takes further products in turn and requests the next one's operands before the
// inverse.  Measured against k_negacyclic_mul<1024>, us per call in a row, operands in the last-level
// cache (3000 products are 37 MB) / streamed through 1.2 GB: 3000 14.1 / 18.7 (2.6 / 2.0 TB/s) against
// 17.9 / 20.5, 4096 19.8 / 21.6 against 23.4 / 25.9, 20,000 78.7 / 84.8 against 92.9 / 97.7; up to 2048
// the host's part of a call, 13.4 either way.  Streamed operands gain less: nothing overlaps the
// first round's loads.  Workgroups of four waves, three per compute unit, each with its own copy
// of the constants and no early requests: 3000 in 20.0 us where this took 15.2.
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_mx_ring(
    MxArgs X, const uint32_t *a, const uint32_t *b, uint32_t *out, size_t count, uint32_t Q, uint32_t qn)
{
    constexpr int REST = MX_VECS - MX_FB * 64, OPS = REST + 16 * 64;  // the block from MX_FB on, then the first stage
    __shared__ v4i area[OPS];
    const v4i *const cst = area - MX_FB * 64, *const fb = area, *const fr = area + REST;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = (lane & 31) + 128 * (lane >> 5);
    const ModS m{(int32_t)Q, qn};
    const size_t waves = blockDim.x >> 6, stride = gridDim.x * waves;
    uint32_t x[2][16];
    auto request = [&](size_t item) {
        const size_t at = (item < count ? item : 0) * MXN + base;
#pragma unroll
        for (int v = 0; v < 16; v++) x[0][v] = a[at + mx_off(v)];
#pragma unroll
        for (int v = 0; v < 16; v++) x[1][v] = b[at + mx_off(v)];
        __builtin_amdgcn_sched_barrier(0);
    };
    request(blockIdx.x * waves + wave);
    mx_copy(OPS, [&](int t) { return reinterpret_cast<const v4i *>(X.cst)[t < REST ? MX_FB * 64 + t : MX_FR - REST + t]; },
            area);
    __syncthreads();
    for (size_t item = blockIdx.x * waves + wave; item < count; item += stride) {
        const size_t at = item * MXN + base;
        int32_t lo[2][16], hi[2][16], ra[16], r4[4];
        v4i z[2][4];
        int64_t s4[4], acc[16];
        // balanced bytes of the centred residue
        auto bytes = [&](int p, int q) {
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const uint32_t t = x[p][4 * q + s] + (Q - 1) / 2;
                z[p][q][s] = (int32_t)((min(t, t - Q) + (BAL - (Q - 1) / 2)) ^ BAL);
            }
        };
#pragma unroll
        for (int q = 0; q < 4; q++) bytes(0, q);
        const v4i *const tw = cst + MX_TWF * 64 + lane;
        mx_stage<false>(fr, z[0], lane, lo[0], hi[0], [&](int t) { if (t & 1) bytes(1, t >> 1); });
        mx_stage<false>(fr, z[1], lane, lo[1], hi[1], [&](int t) { mx_twist(t, lo[0], hi[0], tw, 64, X, m, s4, z[0]); });
        mx_stage<true>(fb, z[0], lane, lo[0], hi[0], [&](int t) { mx_twist(t, lo[1], hi[1], tw, 64, X, m, s4, z[1]); });
        // A 2^-32, then B (2^96 / N) 2^-32: the inverse takes another 2^-32
        mx_stage<true>(fb, z[1], lane, lo[1], hi[1], [&](int t) {
            const int q = t >> 1;
            if (!(t & 1)) {
#pragma unroll
                for (int s = 0; s < 4; s++) s4[s] = (int64_t)hi[0][4 * q + s] * X.two16 + lo[0][4 * q + s];
            } else {
                redc4(s4, m, r4);
#pragma unroll
                for (int s = 0; s < 4; s++) ra[4 * q + s] = r4[s];
            }
        });
#pragma unroll
        for (int q = 0; q < 4; q++) {
#pragma unroll
            for (int s = 0; s < 4; s++) s4[s] = (int64_t)hi[1][4 * q + s] * X.ring16 + (int64_t)lo[1][4 * q + s] * X.ring;
            redc4(s4, m, r4);
#pragma unroll
            for (int s = 0; s < 4; s++) acc[4 * q + s] = (int64_t)ra[4 * q + s] * r4[s];
        }
        request(item + stride < count ? item + stride : item);  // the wave's next product
        mx_inverse_part(acc, cst, lane, X, m, [&](int v, uint32_t c) { out[at + mx_off(v)] = c; });
    }
}

// ------------------------------------------------------------------ one CMux step

// One wave per component; workgroups of eight waves, or of four while that gives every component
// a SIMD of its own (launch_mx_step).
template <int KEYS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_step(WideArgs A, uint32_t num_tasks)
{
    __shared__ v4i cst[MX_VECS];
    __shared__ v4i digits[8][MX_MAX_L * 2 * 64];
    mx_copy<8>(MX_VECS, [&](int t) { return reinterpret_cast<const v4i *>(A.mx.cst)[t]; }, cst);
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t waves = blockDim.x >> 6;
    v4i *const dig = digits[wave];
    const uint32_t Q = A.Q[0];
    const ModS m{(int32_t)Q, A.qn[0]};
    const uint32_t slot = xcd_item(blockIdx.x, gridDim.x) * waves + wave;
    for (uint32_t item = slot; item < num_tasks; item += gridDim.x * waves) {
        const WideTask &T = A.tasks[item];
        const uint32_t i = __builtin_amdgcn_readfirstlane(T.i0) + A.step;
        const uint32_t r = __builtin_amdgcn_readfirstlane(T.r), comp = __builtin_amdgcn_readfirstlane(T.comp);
        const uint32_t q_in = __builtin_amdgcn_readfirstlane(T.q_in);
        const uint32_t *const ct_acc = A.acc_rd + T.acc_off, *const own = ct_acc + (size_t)comp * 2 * MXN;
        uint32_t *const wr = A.acc_wr + T.acc_off + (size_t)comp * 2 * MXN;
        uint32_t base = (lane & 31) + 128 * (lane >> 5);
        __asm__("" : "+v"(base));  // opaque: addresses are formed where they are used
        if (i >= A.n) {
#pragma unroll
            for (int v = 0; v < 16; v++) {
                wr[base + mx_off(v)] = own[base + mx_off(v)];
                wr[base + MXN + mx_off(v)] = own[base + MXN + mx_off(v)];
            }
            continue;
        }
        const uint32_t M = 2u * MXN * r;
        const uint32_t am =
            __builtin_amdgcn_readfirstlane(modswitch_dev(A.ct_in[(size_t)T.ct * A.ct_stride + i], q_in, M));
        int64_t acc[2][16];
#pragma unroll
        for (int v = 0; v < 16; v++) acc[0][v] = acc[1][v] = 0;
#pragma unroll 1
        for (int key = 0; key < KEYS; key++) {
            uint32_t src, e;
            phi_row(key == 0 ? (M - am) % M : am, r, comp, src, e);
            const uint32_t *sp = ct_acc + (size_t)src * 2 * MXN;
            const uint32_t rb = base + 2 * MXN - (e % (2 * MXN));
            // every word is requested before the first is used
            uint32_t vo[2][16], vs[2][16];
#pragma unroll
            for (int p = 0; p < 2; p++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    vo[p][v] = own[base + p * MXN + mx_off(v)];
                    vs[p][v] = sp[p * MXN + ((rb + mx_off(v)) & (MXN - 1))];
                }
            __builtin_amdgcn_sched_barrier(0);
            uint32_t y[2][16];
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const uint32_t flip = 0u - (((rb + mx_off(v)) >> 10) & 1u);
                const uint32_t fq = flip & (Q + 1);
#pragma unroll
                for (int p = 0; p < 2; p++) y[p][v] = mx_field(vs[p][v], vo[p][v], flip, fq, Q, A.mx, A.sg);
            }
            mx_digits<2>(y, A.l, A.log2B, A.mx, lane, dig);
            mx_products(dig, cst, A.mx.bsk + ((size_t)i * KEYS + key) * (4u * A.l * MXN), A.l, lane, A.mx, m, acc);
            if (KEYS == 2 && key == 0) mx_fold(acc, A.mx);
        }
        uint32_t old[2][16];  // this component's accumulator again, requested early
        uint32_t pos = base;
        __asm__("" : "+v"(pos));
#pragma unroll
        for (int p = 0; p < 2; p++)
#pragma unroll
            for (int v = 0; v < 16; v++) old[p][v] = own[pos + p * MXN + mx_off(v)];
        __builtin_amdgcn_sched_barrier(0);
        mx_inverse(acc, cst, lane, A.mx, m,
                   [&](int p, int v, uint32_t x) { wr[pos + p * MXN + mx_off(v)] = add_q(old[p][v], x, Q); });
    }
}

// ------------------------------------------------------------------ two primes, N = 2048
//
// N = 64 x 32: the first stage contracts over i1 < 64 and its outputs k1 fall into T1 = 2 tiles
// of 32, after which everything up to the products is local to a tile; the inverse's last
// stage contracts over all k1 and its outputs i1 fall into two tiles again.  A wave owns one
// tile of one prime of a component, four waves per component.  A digit (at most 15 bits)
// is two balanced bytes; the component's waves form the digits of one part together (each
// wave one of the four contraction blocks) in LDS, and swap tiles through LDS before the
// last stage.
//
// Bound by vector issue and the chain of one wave: with a ternary secret a step of one component
// is some 100k clocks of its four waves (eight pairs of products 47k, digits 15k, the inverse and
// its last stage 15k), and two components share a compute unit's SIMDs.  Measured at n = 512,
// ternary, 2400 components: 138.7 ms, against 195.6 for one butterfly workgroup per component
// and prime.  Of that the requests in groups (the digits' words, the last stage's constants:
// left alone the compiler waits for every few) brought 162 -> 139 ms.

// Operands per prime in LDS: the first stage [tile][block][limb], the second [q][limb], the
// forward twiddles [tile][q][w, 2^16 w]; in memory behind both primes' of them, per prime, the
// inverse twiddles [tile][q][w, 2^16 w] and the last stage [tile out][tile in][q][limb].  The
// second prime is below 2^24: three limbs.
struct MxWide {
    static constexpr int T1 = 2, N = 1024 * T1, NB = 2 * T1, WAVES = 2 * T1, COMPS = 8 / WAVES, E = 8;
    static constexpr int fb(int nl) { return T1 * NB * nl; }
    static constexpr int twf(int nl) { return fb(nl) + 4 * nl; }
    static constexpr int lds_ops(int nl) { return twf(nl) + 8 * T1; }
    static constexpr int IA = 8 * T1;  // behind the inverse twiddles
    static constexpr int LDS_OPS = 7 * (T1 * NB + 4) + 16 * T1;  // lds_ops of both
    static constexpr int mem(int pr) { return LDS_OPS + pr * (IA + 16 * T1 * T1); }
    static_assert((LDS_OPS + 2 * IA + 28 * T1 * T1) * 256 == (int)MX_WIDE_CONST_WORDS, "constant block");
};

// Two digit polynomials (digits u, u + 1 of one part; their blocks at d0, d1) through both
// forward stages and onto acc with their key rows kr[poly] (tile's [part][q][lane]).
template <int NB, int NL>
__device__ __forceinline__ void mx_wide_pair(const v4i *d0, const v4i *d1, const v4i *fa, const v4i *fb, const v4i *tw,
                                              const v4i *const (&kr)[2], size_t part_stride, int lane, const MxArgs &X,
                                              const ModS &m, int64_t (&acc)[2][16])
{
    int32_t lo[2][16], hi[2][16];
    v4i z[2][4], k[2][2][4];
    int64_t s4[4];
    int32_t r4[4];
    auto request = [&](int p) {
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int o = 0; o < 2; o++) k[p][o][q] = kr[p][o * part_stride + q * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int jj = 0; jj < 2; jj++) {
        v16i c[2][2] = {};
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const v4i x[2] = {d0[b * 64 + lane], d1[b * 64 + lane]};
#pragma unroll
            for (int j = 0; j < (jj ? NL - 2 : 2); j++) {
                const v4i w = fa[(NL * b + 2 * jj + j) * 64 + lane];
#pragma unroll
                for (int p = 0; p < 2; p++) c[p][j] = mfma(x[p], w, c[p][j]);
            }
        }
#pragma unroll
        for (int p = 0; p < 2; p++) mx_join<NL>(jj, c[p][0], c[p][1], jj ? hi[p] : lo[p]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < 8; t++) mx_twist(t, lo[0], hi[0], tw + lane, 64, X, m, s4, z[0]);
    request(0);
    mx_stage<true, NL>(fb, z[0], lane, lo[0], hi[0], [&](int t) { mx_twist(t, lo[1], hi[1], tw + lane, 64, X, m, s4, z[1]); });
    request(1);
    mx_stage<true, NL>(fb, z[1], lane, lo[1], hi[1], [&](int t) { mx_mac(t, lo[0], hi[0], k[0], X, m, r4, acc); });
#pragma unroll
    for (int t = 0; t < 8; t++) mx_mac(t, lo[1], hi[1], k[1], X, m, r4, acc);
}

// Digits of contraction block b of one part: element e of a lane is coefficient 32 i1 + col,
// i1 = 16 b + 8 half + e.  Every word (own and rotated source, both primes) is requested
// before the first is used.
struct MxWords {
    uint32_t own[2][8], src[2][8];
};

__device__ __forceinline__ uint32_t mx_wide_at(int b, int lane) { return 32 * (16 * b + 8 * (lane >> 5)) + (lane & 31); }

__device__ __forceinline__ void mx_wide_request(MxWords &d, const uint32_t *own, const uint32_t *src, const WideRow &w,
                                                int b, int lane)
{
    constexpr int N = MxWide::N;
    const uint32_t at = mx_wide_at(b, lane);
#pragma unroll
    for (int p = 0; p < 2; p++)
#pragma unroll
        for (int e = 0; e < 8; e++) {
            d.own[p][e] = own[p * N + at + 32 * e];
            d.src[p][e] = src[p * N + ((at + 32 * e - w.e) & (N - 1))];
        }
}

__device__ __forceinline__ void mx_wide_digits(const MxWords &d, const WideRow &w, int b, const WideArgs &A, int lane,
                                               v4i *dig)
{
    constexpr int NB = MxWide::NB;
    const uint32_t at = mx_wide_at(b, lane);
    const ModQ m1{A.Q[1], A.qn[1]};
    const uint64_t hw = (A.Qw - 1) / 2;
    uint64_t y[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const bool flip = (at + 32 * e < w.e) != w.neg;
        auto diff = [&](int p) {
            const uint32_t v = d.src[p][e], Q = A.Q[p];
            return sub_q(flip && v ? Q - v : v, d.own[p][e], Q);
        };
        const uint32_t a0 = diff(0), a1 = diff(1);
        // x = a0 + Q0 ((a1 - a0) Q0^-1 mod Q1), in [0, Q0 Q1)
        const uint64_t x = a0 + (uint64_t)A.Q[0] * mont_mul(a1 + A.crt_cq - a0, A.crt_inv, m1);
        int64_t xc = x > hw ? (int64_t)(x - A.Qw) : (int64_t)x;
        if (A.sg) xc = (xc + (1ll << (A.sg - 1))) >> A.sg;
        y[e] = (uint64_t)xc + A.goff;
    }
    for (uint32_t u = 0; u < A.l; u++) {
        const uint32_t sh = u * A.log2B;
        const uint32_t mask = u + 1 == A.l ? 0xffffu : (1u << A.log2B) - 1;
        v4i x;
#pragma unroll
        for (int g = 0; g < 4; g++) {
            // two fields, minus B/2, as two balanced bytes each: + 0x80, low byte xor 0x80
            const uint32_t f0 = ((uint32_t)(y[2 * g] >> sh) & mask) + A.mx.bias16;
            const uint32_t f1 = ((uint32_t)(y[2 * g + 1] >> sh) & mask) + A.mx.bias16;
            x[g] = (int32_t)(((f0 & 0xffffu) | (f1 << 16)) ^ 0x00800080u);
        }
        dig[(u * NB + b) * 64 + lane] = x;
    }
    if (A.l & 1) dig[(A.l * NB + b) * 64 + lane] = v4i{};  // the last pair's second polynomial
}

// The last inverse stage of one prime for output tile `tile` of P parts: z(p, block) the tiles'
// values as operands, ia the tile's constants in memory.  Constants in groups of four blocks,
// each group requested before the one in hand is used.
template <int P, int NL, class Z>
__device__ __forceinline__ void mx_wide_last(const v4i *ia, uint32_t pos, Z z, int32_t (&lo)[P][16], int32_t (&hi)[P][16])
{
    constexpr int T1 = MxWide::T1;
    v4i kc[2][8];
    auto request = [&](int g) {
        const int jj = g / T1;
#pragma unroll
        for (int b = 0; b < 4; b++)
#pragma unroll
            for (int j = 0; j < (jj ? NL - 2 : 2); j++)
                kc[g & 1][2 * b + j] = ia[(NL * (4 * (g % T1) + b) + 2 * jj + j) * 64 + pos];
        __builtin_amdgcn_sched_barrier(0);
    };
    request(0);
    v16i c[P][2];
#pragma unroll
    for (int g = 0; g < 2 * T1; g++) {
        const int jj = g / T1;
        if (g + 1 < 2 * T1) request(g + 1);
        if (g % T1 == 0) {
#pragma unroll
            for (int p = 0; p < P; p++) c[p][0] = c[p][1] = v16i{};
        }
#pragma unroll
        for (int b = 0; b < 4; b++) {
            v4i x[P];
#pragma unroll
            for (int p = 0; p < P; p++) x[p] = z(p, 4 * (g % T1) + b);
#pragma unroll
            for (int j = 0; j < (jj ? NL - 2 : 2); j++)
#pragma unroll
                for (int p = 0; p < P; p++) c[p][j] = mfma(kc[g & 1][2 * b + j], x[p], c[p][j]);
        }
        if (g % T1 == T1 - 1) {
#pragma unroll
            for (int p = 0; p < P; p++) mx_join<NL>(jj, c[p][0], c[p][1], jj ? hi[p] : lo[p]);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// to = from + the coefficients lo + 2^16 hi of one part and tile (to and from at the tile).
__device__ __forceinline__ void mx_wide_store(const uint32_t *from, uint32_t *to, uint32_t pos, const int32_t (&lo)[16],
                                              const int32_t (&hi)[16], int32_t two32, int32_t two48, const ModS &m)
{
    const uint32_t at = 128 * (pos >> 5) + (pos & 31), Q = (uint32_t)m.Q;
    uint32_t old[16];
#pragma unroll
    for (int v = 0; v < 16; v++) old[v] = from[at + mx_off(v)];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        int64_t s4[4];
        int32_t o[4];
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] = (int64_t)lo[4 * q + s] * two32 + (int64_t)hi[4 * q + s] * two48;
        redc4(s4, m, o);
#pragma unroll
        for (int s = 0; s < 4; s++)  // o in (-Q, Q)
            to[at + mx_off(4 * q + s)] = add_q(old[4 * q + s], min((uint32_t)o[s], (uint32_t)o[s] + Q), Q);
    }
}

// A barrier among the waves of one component: the other components of the workgroup go
// their own pace, so that one's digits (memory latency, vector work) run beside another's
// products.  Every wave of the component arrives, all are resident: the wait ends.
struct CompSync {
    uint32_t *count;
    uint32_t target, waves;
    __device__ __forceinline__ void wait_for(const uint32_t *c, uint32_t t) const
    {
        while ((int32_t)(__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - t) < 0)
            __builtin_amdgcn_s_sleep(1);
    }
    __device__ __forceinline__ void operator()()
    {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        target += waves;
        wait_for(count, target);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
};

// One step of the components of a workgroup for a wave of prime pr (NL limbs); constants,
// digits (and, before the last stage, the tiles the component's waves swap) in LDS.
template <int KEYS, int NL>
__device__ __forceinline__ void mx_wide_run(const WideArgs &A, uint32_t num_tasks, const v4i *cst, v4i *digits,
                                             uint32_t *arrive)
{
    using C = MxWide;
    constexpr int T1 = C::T1, N = C::N, NB = C::NB, E = C::E;
    constexpr int pr = NL == 3 ? 1 : 0;
    constexpr size_t PW = (size_t)2 * N, CW = 2 * PW;  // words per part, per component
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int cw = wave / C::WAVES, wi = wave % C::WAVES, tile = wi % T1;
    v4i *const dig = digits + cw * MX_MAX_L * NB * 64;
    const v4i *const base = cst + (pr ? C::lds_ops(4) * 64 : 0), *const fb = base + C::fb(NL) * 64;
    const v4i *const mem = reinterpret_cast<const v4i *>(A.mx.cst) + (size_t)C::mem(pr) * 64;
    const uint32_t Q = A.Q[pr];
    const ModS m{(int32_t)Q, A.qn[pr]};
    MxArgs X = A.mx;
    X.two32 = pr ? A.mx.two32_1 : A.mx.two32;
    const int32_t two48 = pr ? A.mx.two48_1 : A.mx.two48;
    const int neg = ((32 - lane) & 31) | (lane & 32);
    const uint32_t pairs = (A.l + 1) / 2;
    CompSync sync{arrive + cw, 0, C::WAVES};
    // the second wave of a SIMD starts when the first one's first digits are written
    if (wave >= 4) sync.wait_for(arrive + (wave - 4) / C::WAVES, 2 * C::WAVES);
    for (uint32_t first = xcd_item(blockIdx.x, gridDim.x) * C::COMPS; first < num_tasks; first += gridDim.x * C::COMPS) {
        const bool has = first + cw < num_tasks;
        const WideTask &T = A.tasks[has ? first + cw : first];
        const uint32_t i = __builtin_amdgcn_readfirstlane(T.i0) + A.step;
        const uint32_t r = __builtin_amdgcn_readfirstlane(T.r), comp = __builtin_amdgcn_readfirstlane(T.comp);
        const uint32_t q_in = __builtin_amdgcn_readfirstlane(T.q_in);
        const bool active = has && i < A.n;
        const uint32_t *const ct_acc = A.acc_rd + T.acc_off, *const own = ct_acc + (size_t)comp * CW;
        uint32_t *const wr = A.acc_wr + T.acc_off + (size_t)comp * CW;
        if (has && !active)  // past step n - 1: carried over
            for (int w = wi * 64 + lane; w < (int)CW; w += 64 * C::WAVES) wr[w] = own[w];
        const uint32_t M = 2u * N * r;
        const uint32_t am =
            active ? __builtin_amdgcn_readfirstlane(modswitch_dev(A.ct_in[(size_t)T.ct * A.ct_stride + i], q_in, M)) : 0u;
        int64_t acc[2][16];
        uint32_t touched = 0;
#pragma unroll
        for (int v = 0; v < 16; v++) acc[0][v] = acc[1][v] = 0;
#pragma unroll 1
        for (int kp = 0; kp < 2 * KEYS; kp++) {
            const int key = kp >> 1, part = kp & 1;
            __asm__ volatile("" ::"v"(touched));
            sync();  // the previous digits (at first: tiles) are read
            if (active) {
                MxWords wd;
                const WideRow w = wide_row(key == 0 ? (M - am) % M : am, r, comp, N);
                mx_wide_request(wd, own + part * PW, ct_acc + (size_t)w.src * CW + part * PW, w, wi, lane);
                __builtin_amdgcn_sched_barrier(0);
                mx_wide_digits(wd, w, wi, A, lane, dig);
            }
            sync();  // the digits are written
            if (active) {
                if (kp + 1 < 2 * KEYS) {
                    // the lines of the next digits' reads, one a lane, so that these find them in L2
                    const WideRow w = wide_row((kp + 1) >> 1 ? am : (M - am) % M, r, comp, N);
                    const uint32_t idx = 32 * (16 * wi + (lane & 15)) + ((lane >> 4) & 1) * N;
                    const uint32_t at = lane < 32 ? idx : (idx & ~(uint32_t)(N - 1)) | ((idx - w.e) & (N - 1));
                    touched = ct_acc[(lane < 32 ? comp : w.src) * CW + ((kp + 1) & 1) * PW + at];
                }
                // digits of a (part 0) meet rows l + u, digits of b rows u (eq. def:gsw)
                const v4i *K = reinterpret_cast<const v4i *>(A.mx.bsk) +
                               (((size_t)i * KEYS + key) * 2 + pr) * (A.l * N) + (size_t)(part ? 0 : A.l) * (N / 2) +
                               tile * 256;
#pragma unroll 1
                for (uint32_t g = 0; g < pairs; g++) {
                    __asm__ volatile("" ::: "memory");
                    const uint32_t u1 = min(2 * g + 1, A.l - 1);  // (its digits are zeros where it repeats a row)
                    const v4i *const kr[2] = {K + (size_t)(2 * g) * (N / 2), K + (size_t)u1 * (N / 2)};
                    mx_wide_pair<NB, NL>(dig + 2 * g * NB * 64, dig + (2 * g + 1) * NB * 64, base + tile * NB * NL * 64,
                                          fb, base + (C::twf(NL) + 8 * tile) * 64, kr, N / 4, lane, X, m, acc);
                }
                if (KEYS == 2 && kp == 1) mx_fold(acc, X);
            }
        }
        // the sums back to coefficients: second stage and twiddles within the tile
        int32_t lo[2][16], hi[2][16];
        v4i z[2][4], ti[8], x0[4 * T1];
        int64_t s4[4];
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < 8; j++) ti[j] = mem[(8 * tile + j) * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; q++) mx_cut(q, acc[0], X, m, s4, z[0]);
        mx_stage<false, NL>(fb, z[0], neg, lo[0], hi[0],
                            [&](int t) { if (t & 1) mx_cut(t >> 1, acc[1], X, m, s4, z[1]); });
        mx_stage<false, NL>(fb, z[1], neg, lo[1], hi[1],
                            [&](int t) { mx_twist(t, lo[0], hi[0], ti, 1, X, m, s4, z[0]); });
#pragma unroll
        for (int t = 0; t < 8; t++) mx_twist(t, lo[1], hi[1], ti, 1, X, m, s4, z[1]);
        // the last stage over all tiles of the prime: the tiles of part 0 into registers, those
        // of part 1 read from LDS as operands, so that both parts share each constant
        v4i *const swap = digits + (wave - tile) * 4 * 64;
        sync();  // the digits are read
#pragma unroll
        for (int q = 0; q < 4; q++) swap[(4 * tile + q) * 64 + lane] = z[0][q];
        sync();
#pragma unroll
        for (int b = 0; b < 4 * T1; b++) x0[b] = swap[b * 64 + lane];
        sync();
#pragma unroll
        for (int q = 0; q < 4; q++) swap[(4 * tile + q) * 64 + lane] = z[1][q];
        sync();
        if (!active) continue;
        uint32_t pos = lane;  // opaque: the addresses below are not carried through the products
        __asm__("" : "+v"(pos));
        const v4i *const ia = mem + (C::IA + 4 * NL * T1 * tile) * 64;
        mx_wide_last<2, NL>(ia, pos, [&](int p, int b) { return p ? swap[b * 64 + lane] : x0[b]; }, lo, hi);
#pragma unroll
        for (int part = 0; part < 2; part++) {
            const size_t at = part * PW + pr * N + 1024 * tile;
            mx_wide_store(own + at, wr + at, pos, lo[part], hi[part], X.two32, two48, m);
        }
    }
}

template <int KEYS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_wide_step(WideArgs A, uint32_t num_tasks)
{
    using C = MxWide;
    __shared__ v4i cst[C::LDS_OPS * 64];
    __shared__ v4i digits[C::COMPS * MX_MAX_L * C::NB * 64];
    __shared__ uint32_t arrive[C::COMPS];
    static_assert(sizeof(digits) == 8 * 4 * 64 * 16, "one part's tile per wave");
    if (threadIdx.x < C::COMPS) arrive[threadIdx.x] = 0;
    mx_copy<8>(C::LDS_OPS * 64, [&](int t) { return reinterpret_cast<const v4i *>(A.mx.cst)[t]; }, cst);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % C::WAVES >= C::T1)
        mx_wide_run<KEYS, 3>(A, num_tasks, cst, digits, arrive);
    else
        mx_wide_run<KEYS, 4>(A, num_tasks, cst, digits, arrive);
}

// Light work: one workgroup per component and prime (work item 2 task + prime), eight waves.
// Wave (g, part, tile): with a ternary secret g is the key, else every other pair of digits; it
// forms KEYS of the part's contraction blocks of the digits, runs its pairs onto both parts'
// sums of its tile, and the sums meet in the waves g = 0, which run the inverse of
// their part and tile.  LDS: one prime's constants, the digits of every key and part, and in
// their place the sums and the tiles.
//
// Bound by the chain of one step (about 13 us of digits, two pairs of products, three
// exchanges and the inverse, 6 of launch): at n = 512, ternary, 16 components take 9.5 ms and 128 9.9,
// against 17.6 for the butterfly workgroups of two digit groups (35 us a step) and 26.3 for four
// waves per component.
template <int KEYS, int NL>
__device__ __forceinline__ void mx_wide_split_run(const WideArgs &A, const WideTask &T, const v4i *cst, v4i *area)
{
    using C = MxWide;
    constexpr int T1 = C::T1, N = C::N, NB = C::NB, pr = NL == 3 ? 1 : 0;
    constexpr size_t PW = (size_t)2 * N, CW = 2 * PW;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = wave >> 2, part = (wave >> 1) & 1, tile = wave & 1;
    const uint32_t i = T.i0 + A.step, r = T.r, comp = T.comp;
    const uint32_t *const ct_acc = A.acc_rd + T.acc_off, *const own = ct_acc + (size_t)comp * CW;
    uint32_t *const wr = A.acc_wr + T.acc_off + (size_t)comp * CW;
    const ModS m{(int32_t)A.Q[pr], A.qn[pr]};
    MxArgs X = A.mx;
    X.two32 = pr ? A.mx.two32_1 : A.mx.two32;
    const int neg = ((32 - lane) & 31) | (lane & 32);
    const int key = KEYS == 2 ? g : 0;
    v4i *const dig = area + (2 * key + part) * MX_MAX_L * NB * 64;
    {
        const uint32_t M = 2u * N * r;
        const uint32_t am =
            __builtin_amdgcn_readfirstlane(modswitch_dev(A.ct_in[(size_t)T.ct * A.ct_stride + i], T.q_in, M));
        const WideRow w = wide_row(key == 0 ? (M - am) % M : am, r, comp, N);
        const uint32_t *const src = ct_acc + (size_t)w.src * CW + part * PW;
        MxWords wd[KEYS];
#pragma unroll
        for (int j = 0; j < KEYS; j++) mx_wide_request(wd[j], own + part * PW, src, w, KEYS == 2 ? 2 * tile + j : 2 * tile + g, lane);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < KEYS; j++) mx_wide_digits(wd[j], w, KEYS == 2 ? 2 * tile + j : 2 * tile + g, A, lane, dig);
    }
    __syncthreads();  // digits and constants are written
    int64_t acc[2][16];
#pragma unroll
    for (int v = 0; v < 16; v++) acc[0][v] = acc[1][v] = 0;
    const uint32_t pairs = (A.l + 1) / 2;
    const v4i *K = reinterpret_cast<const v4i *>(A.mx.bsk) + (((size_t)i * KEYS + key) * 2 + pr) * (A.l * N) +
                   (size_t)(part ? 0 : A.l) * (N / 2) + tile * 256;
#pragma unroll 1
    for (uint32_t k = KEYS == 2 ? 0 : g; k < pairs; k += KEYS == 2 ? 1 : 2) {
        __asm__ volatile("" ::: "memory");
        const uint32_t u1 = min(2 * k + 1, A.l - 1);
        const v4i *const kr[2] = {K + (size_t)(2 * k) * (N / 2), K + (size_t)u1 * (N / 2)};
        mx_wide_pair<NB, NL>(dig + 2 * k * NB * 64, dig + (2 * k + 1) * NB * 64, cst + tile * NB * NL * 64,
                             cst + C::fb(NL) * 64, cst + (C::twf(NL) + 8 * tile) * 64, kr, N / 4, lane, X, m, acc);
    }
    mx_fold(acc, X);  // four waves' sums of up to four products each then stay below 2^63
    auto send = [&](v4i *to, const int64_t (&t)[16]) {
#pragma unroll
        for (int v = 0; v < 8; v++)
            to[v * 64 + lane] = v4i{(int32_t)t[2 * v], (int32_t)(t[2 * v] >> 32), (int32_t)t[2 * v + 1],
                                    (int32_t)(t[2 * v + 1] >> 32)};
    };
    auto receive = [&](const v4i *from, int64_t (&t)[16]) {
#pragma unroll
        for (int v = 0; v < 8; v++) {
            const v4i x = from[v * 64 + lane];
            t[2 * v] += (int64_t)((uint64_t)(uint32_t)x[1] << 32 | (uint32_t)x[0]);
            t[2 * v + 1] += (int64_t)((uint64_t)(uint32_t)x[3] << 32 | (uint32_t)x[2]);
        }
    };
    __syncthreads();  // the digits are read
    if (g == 1) {
        send(area + (wave & 3) * 1024, acc[0]);
        send(area + (wave & 3) * 1024 + 512, acc[1]);
    }
    __syncthreads();
    int64_t sum[16];
    if (g == 0) {
        receive(area + wave * 1024, acc[0]);
        receive(area + wave * 1024 + 512, acc[1]);
        __asm__ volatile("" ::: "memory");
#pragma unroll
        for (int v = 0; v < 16; v++) {
            sum[v] = part ? acc[1][v] : acc[0][v];
            acc[0][v] = part ? acc[0][v] : acc[1][v];
        }
        send(area + wave * 1024, acc[0]);  // the other part's, in the place this wave alone has read
    }
    __syncthreads();
    int32_t lo[1][16], hi[1][16];
    v4i z[4];
    const v4i *const mem = reinterpret_cast<const v4i *>(A.mx.cst) + (size_t)C::mem(pr) * 64;
    if (g == 0) {
        receive(area + (wave ^ 2) * 1024, sum);
        int64_t s4[4];
        v4i ti[8];
#pragma unroll
        for (int j = 0; j < 8; j++) ti[j] = mem[(8 * tile + j) * 64 + lane];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; q++) mx_cut(q, sum, X, m, s4, z);
        mx_stage<false, NL>(cst + C::fb(NL) * 64, z, neg, lo[0], hi[0], [](int) {});
#pragma unroll
        for (int t = 0; t < 8; t++) mx_twist(t, lo[0], hi[0], ti, 1, X, m, s4, z);
    }
    __syncthreads();  // the sums are read
    v4i *const tiles = area + part * 8 * 64;
    if (g == 0) {
#pragma unroll
        for (int q = 0; q < 4; q++) tiles[(4 * tile + q) * 64 + lane] = z[q];
    }
    __syncthreads();
    if (g == 1) return;
    uint32_t pos = lane;
    __asm__("" : "+v"(pos));
    mx_wide_last<1, NL>(mem + (C::IA + 4 * NL * T1 * tile) * 64, pos, [&](int, int b) { return tiles[b * 64 + lane]; }, lo, hi);
    const size_t at = part * PW + pr * N + 1024 * tile;
    mx_wide_store(own + at, wr + at, pos, lo[0], hi[0], X.two32, pr ? A.mx.two48_1 : A.mx.two48, m);
}

template <int KEYS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_wide_split(WideArgs A)
{
    using C = MxWide;
    __shared__ v4i cst[C::lds_ops(4) * 64];
    __shared__ v4i area[4 * 1024];  // digits [key][part][u][block], then sums, then tiles
    static_assert(2 * 2 * MX_MAX_L * C::NB * 64 <= 4 * 1024, "digits of two keys");
    const uint32_t item = xcd_item(blockIdx.x, gridDim.x);
    const WideTask T = A.tasks[item / 2];
    const int pr = item & 1;
    if (T.i0 + A.step >= A.n) {  // past step n - 1: carried over
        const size_t off = T.acc_off + (size_t)T.comp * 4 * C::N + (size_t)pr * C::N;
        for (uint32_t w = threadIdx.x; w < 2u * C::N; w += 512) {
            const size_t at = off + (size_t)(w / C::N) * 2 * C::N + w % C::N;
            A.acc_wr[at] = A.acc_rd[at];
        }
        return;
    }
    const v4i *src = reinterpret_cast<const v4i *>(A.mx.cst) + (pr ? C::lds_ops(4) * 64 : 0);
    const int ops = pr ? C::lds_ops(3) : C::lds_ops(4);
    mx_copy<8>(ops * 64, [&](int t) { return src[t]; }, cst);
    if (pr) mx_wide_split_run<KEYS, 3>(A, T, cst, area);
    else mx_wide_split_run<KEYS, 4>(A, T, cst, area);
}

// The bootstrapping key in these kernels' order: dst[poly][tile][q][lane][s], entry of
// NTT position k = k1 + 32 T1 k2 (k1 = 32 tile + lane % 32, k2 = 8 q + 4 (lane / 32) + s), from
// the bit-reversed, Montgomery-form key, times another 2^32 and balanced.  The polynomials
// of prime pr are blocks of `block` every primes * block.
__global__ __launch_bounds__(256) void k_mx_keys(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst, int logN,
                                                 uint32_t Q, uint32_t qn, uint32_t two64, uint32_t block, uint32_t primes,
                                                 uint32_t pr)
{
    const uint32_t N = 1u << logN, b = blockIdx.x / block;
    const size_t base = ((size_t)(b * primes + pr) * block + blockIdx.x % block) * N;
    const ModQ m{Q, qn};
    for (uint32_t t = threadIdx.x; t < N; t += 256) {
        const uint32_t tile = t >> 10, q = (t >> 8) & 3, lane = (t >> 2) & 63, s = t & 3;
        const uint32_t k = 32 * tile + (lane & 31) + (N / 32) * (8 * q + 4 * (lane >> 5) + s);
        const uint32_t x = mont_mul(src[base + (__brev(k) >> (32 - logN))], two64, m);
        dst[base + t] = x > (Q - 1) / 2 ? x - Q : x;
    }
}

void launch_mx_keys(uint32_t N, const uint32_t *src, uint32_t *dst, size_t polys, uint32_t Q, uint32_t qn, uint32_t two64,
                    uint32_t block, uint32_t primes, uint32_t pr, hipStream_t st)
{
    int logN = 0;
    while ((1u << logN) < N) logN++;
    hipLaunchKernelGGL(k_mx_keys, dim3((uint32_t)polys), dim3(256), 0, st, src, dst, logN, Q, qn, two64, block, primes, pr);
}

void launch_mx_rotate(const BrArgs &A, int grid, hipStream_t st, int wpp)
{
#define R_(w)                                                                                \
    if (A.keys == 2) hipLaunchKernelGGL((k_mx_rotate<2, w>), dim3(grid), dim3(512), 0, st, A); \
    else hipLaunchKernelGGL((k_mx_rotate<1, w>), dim3(grid), dim3(512), 0, st, A)
    if (wpp == 2) {
        R_(2);
    } else {
        R_(1);
    }
#undef R_
}

void launch_mx_step(uint32_t N, int npr, uint32_t keys, const WideArgs &A, uint32_t num_tasks, hipStream_t st)
{
    if (npr == 2 && N == 2048) {
        const uint32_t grid = std::min<uint32_t>((num_tasks + MxWide::COMPS - 1) / MxWide::COMPS, A.mx.num_cu);
        if (keys == 2) hipLaunchKernelGGL(k_mx_wide_step<2>, dim3(grid), dim3(512), 0, st, A, num_tasks);
        else hipLaunchKernelGGL(k_mx_wide_step<1>, dim3(grid), dim3(512), 0, st, A, num_tasks);
        return;
    }
    if (npr != 1 || N != 1024) return;
    const uint32_t waves = num_tasks <= 4 * A.mx.num_cu ? 4 : 8;
    const uint32_t grid = std::min<uint32_t>((num_tasks + waves - 1) / waves, A.mx.num_cu);
    if (keys == 2) hipLaunchKernelGGL(k_mx_step<2>, dim3(grid), dim3(64 * waves), 0, st, A, num_tasks);
    else hipLaunchKernelGGL(k_mx_step<1>, dim3(grid), dim3(64 * waves), 0, st, A, num_tasks);
}

void launch_mx_product(const MxArgs &X, const uint32_t *in, uint32_t *out, size_t count, uint32_t key, uint32_t Q,
                       uint32_t qn, uint32_t log2B, uint32_t l, uint32_t sg, hipStream_t st)
{
    // two waves per pair while one round of workgroups (one per compute unit) takes them all: 1024
    // pairs 13.4 us; the next pair would cost a second round, 1025 pairs take 20.5 us with one
    const bool two = count <= 4 * X.num_cu;
    const dim3 grid((uint32_t)((count + 3) / 4));
    if (two) hipLaunchKernelGGL(k_mx_product<2>, grid, dim3(512), 0, st, X, in, out, count, key, Q, qn, log2B, l, sg);
    else hipLaunchKernelGGL(k_mx_product<1>, grid, dim3(256), 0, st, X, in, out, count, key, Q, qn, log2B, l, sg);
}

void launch_mx_ring(const MxArgs &X, const uint32_t *a, const uint32_t *b, uint32_t *out, size_t count, uint32_t Q,
                    uint32_t qn, hipStream_t st)
{
    // up to twelve waves per compute unit (three per SIMD) in as few rounds of equal size (4096 products
    // 21.5 us in two rounds of eight, 26.5 in rounds of twelve); at least four, which fetch the constants together
    const size_t per_cu = (count + X.num_cu - 1) / X.num_cu, rounds = (per_cu + 11) / 12;
    const uint32_t waves = (uint32_t)std::max<size_t>((per_cu + rounds - 1) / rounds, 4);
    const uint32_t grid = (uint32_t)std::min<size_t>((count + waves - 1) / waves, X.num_cu);
    hipLaunchKernelGGL(k_mx_ring, dim3(grid), dim3(64 * waves), 0, st, X, a, b, out, count, Q, qn);
}

void launch_mx_split(uint32_t keys, const WideArgs &A, uint32_t num_tasks, hipStream_t st)
{
    if (keys == 2) hipLaunchKernelGGL(k_mx_wide_split<2>, dim3(2 * num_tasks), dim3(512), 0, st, A);
    else hipLaunchKernelGGL(k_mx_wide_split<1>, dim3(2 * num_tasks), dim3(512), 0, st, A);
}

bool mx_supports(uint32_t N, int npr) { return N == (npr == 2 ? 2048u : 1024u); }

}  // namespace dev
}  // namespace mm
