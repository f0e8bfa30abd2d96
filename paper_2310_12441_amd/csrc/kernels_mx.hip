// The CMux step on the matrix cores (one prime below 2^31, N = 1024).
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

#include "device_common.hpp"
#include "kernels.hpp"
#include "rotation_common.hpp"

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
    for (int s = 0; s < 4; s++) o[s] = (int32_t)((t[s] + (int64_t)q[s] * m.Q) >> 32);
}

__device__ __forceinline__ v16i mfma(v4i a, v4i b, v16i c) { return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0); }

// The constant block (mx_tables in device.cpp), operands of 64 lanes x 16 bytes: the first
// stage's four limbs, the second stage's [contraction block][limb], the forward twiddles
// [block][w, 2^16 w], the last inverse stage's row factors [block][lane half][f, 2^16 f]
// -- these in LDS -- and the inverse twiddles, read once per step from memory.  The inverse
// stages use the second stage's matrix at the negated column (w^(-a b) = w^(a (32 - b))).
enum { MX_FA = 0, MX_FB = 4, MX_TWF = 20, MX_FIN = 28 };
constexpr int MX_VECS = MX_FIN * 64 + 16;
static_assert((MX_VECS + 8 * 64) * 4 == (int)MX_CONST_WORDS, "constant block size");

// Position of register v of a lane: row 8 (v / 4) + 4 half + v % 4, 32 words per row.
__device__ __forceinline__ int mx_off(int v) { return 256 * (v / 4) + 32 * (v % 4); }

// One 32-point stage on a residue polynomial given as bytes: the four limb sums of each
// output joined to lo + 2^16 hi, two limbs at a time.  LEFT: the constant is the left
// operand.  work(t), t = 0 .. 7, is vector arithmetic of another polynomial placed after
// every second instruction: alone, a wave's matrix instructions would leave the vector
// ALU idle and its arithmetic the matrix unit (40 matrix instructions and 480 others of
// this mix take 3.7k clocks per wave one after the other, 3.2k interleaved, at two waves
// per SIMD).
template <bool LEFT, class Work>
__device__ __forceinline__ void mx_stage(const v4i *cst, const v4i (&z)[4], int lane, int32_t (&lo)[16],
                                         int32_t (&hi)[16], Work work)
{
    v4i k[2] = {cst[MX_FB * 64 + lane], cst[(MX_FB + 1) * 64 + lane]};
    v16i c[2];
#pragma unroll
    for (int t = 0; t < 8; t++) {
        const int q = t & 3;
        if (q == 0) c[0] = c[1] = v16i{};
#pragma unroll
        for (int j = 0; j < 2; j++) c[j] = LEFT ? mfma(k[j], z[q], c[j]) : mfma(z[q], k[j], c[j]);
        if (t < 7) {
#pragma unroll
            for (int j = 0; j < 2; j++) k[j] = cst[(MX_FB + 4 * ((t + 1) & 3) + 2 * ((t + 1) >> 2) + j) * 64 + lane];
        }
        work(t);
        if (q == 3) {
#pragma unroll
            for (int v = 0; v < 16; v++) (t == 7 ? hi : lo)[v] = c[0][v] + (int32_t)((uint32_t)c[1][v] << 8);
        }
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
        for (int s = 0; s < 4; s++) s4[s] = (int64_t)hi[4 * q + s] * w16[s] + X.bal64;
#pragma unroll
        for (int s = 0; s < 4; s++) s4[s] += (int64_t)lo[4 * q + s] * w[s];
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

// Digit u of the fields y of both parts as signed bytes, the first stage's operand, into
// the wave's LDS (each lane reads back only its own).
__device__ __forceinline__ void mx_digits(const uint32_t (&y)[2][16], uint32_t l, uint32_t log2B, const MxArgs &X,
                                          int lane, v4i *dig)
{
#pragma unroll
    for (uint32_t u = 0; u < MX_MAX_L; u++) {
        if (u >= l) break;
        const uint32_t sh = u * log2B, wd = log2B + (u + 1 == l ? 1u : 0u);
#pragma unroll
        for (int part = 0; part < 2; part++) {
            v4i d;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                uint32_t p = 0;
#pragma unroll
                for (int s = 0; s < 4; s++) p |= __builtin_amdgcn_ubfe(y[part][4 * q + s], sh, wd) << (8 * s);
                d[q] = (int32_t)((p + X.bias) ^ BAL);
            }
            dig[(2 * u + part) * 64 + lane] = d;
        }
    }
}

// acc += the digit polynomials times their key rows: digits of a (part 0) meet rows l + u,
// digits of b rows u (eq. def:gsw).
__device__ __forceinline__ void mx_products(const v4i *dig, const v4i *cst, const int32_t *K, uint32_t l, int lane,
                                            const MxArgs &X, const ModS &m, int64_t (&acc)[2][16])
{
    for (uint32_t u = 0; u < l; u++) {
        __asm__ volatile("" ::: "memory");  // constants and key words are read where they are used
        int32_t lo[2][16], hi[2][16];
        v4i z[2][4], k[2][2][4];
        int64_t s4[4];
        int32_t r4[4];
        auto request = [&](int p) {
            const v4i *kr = reinterpret_cast<const v4i *>(K + (size_t)(p ? u : l + u) * 2 * MXN) + lane;
#pragma unroll
            for (int q = 0; q < 4; q++)
#pragma unroll
                for (int o = 0; o < 2; o++) k[p][o][q] = kr[(4 * o + q) * 64];
            __builtin_amdgcn_sched_barrier(0);
        };
        const v4i x[2] = {dig[2 * u * 64 + lane], dig[(2 * u + 1) * 64 + lane]};
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
        mx_stage<true>(cst, z[0], lane, lo[0], hi[0],
                       [&](int t) { mx_twist(t, lo[1], hi[1], cst + MX_TWF * 64 + lane, 64, X, m, s4, z[1]); });
        request(1);
        mx_stage<true>(cst, z[1], lane, lo[1], hi[1], [&](int t) { mx_mac(t, lo[0], hi[0], k[0], X, m, r4, acc); });
#pragma unroll
        for (int t = 0; t < 8; t++) mx_mac(t, lo[1], hi[1], k[1], X, m, r4, acc);
    }
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
    auto cut = [&](int p, int q) {
        // 2^32 h + l -> h (2^32 mod Q) + l, which one reduction brings below 2^31; BAL as its bias
        int32_t o[4];
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const uint64_t low = (uint32_t)acc[p][4 * q + s] | ((uint64_t)BAL << 32);
            s4[s] = (int64_t)(int32_t)(acc[p][4 * q + s] >> 32) * X.two32 + (int64_t)low;
        }
        redc4(s4, m, o);
#pragma unroll
        for (int s = 0; s < 4; s++) z[p][q][s] = o[s] ^ (int32_t)BAL;
    };
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
    mx_stage<false>(cst, z[0], neg, lo[0], hi[0], [&](int t) { if (t & 1) cut(1, t >> 1); });
    mx_stage<false>(cst, z[1], neg, lo[1], hi[1], [&](int t) { twist(0, t); });
    mx_stage<true>(cst, z[0], neg, lo[0], hi[0], [&](int t) { twist(1, t); });
    mx_stage<true>(cst, z[1], neg, lo[1], hi[1], [&](int t) { if (t & 1) last(0, t >> 1); });
#pragma unroll
    for (int q = 0; q < 4; q++) last(1, q);
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

// All n CMux steps of up to eight ring components per workgroup, one wave per component
// (the groups and tasks of k_blind_rotate): the accumulators stay in LDS, one buffer,
// two workgroup barriers per step (every rotation has read; every component is written).
//
// Bound by vector issue: a component's step is 3,440 vector and 224 matrix instructions
// (71 % of the four-clock issue slots; the matrix unit is busy 34 % of the time and each of
// its instructions holds vector issue for about 12 clocks), at the 2.0 GHz the device runs
// under this load.  Two waves per SIMD: 256 registers hold the 64-bit sums (64), two
// polynomials' values and the key words in flight; LDS holds the constants (29 KB), the
// digits (64 KB) and the accumulators (64 KB) of eight waves.  Measured for 16,384 components,
// 630 steps: 102 ms, against 183 for k_wide_step<1024, 1, 1, 4> and 204 for k_blind_rotate;
// one workgroup alone 7.4 ms with one wave per SIMD, 12.8 with two.
template <int KEYS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_rotate(BrArgs A)
{
    __shared__ v4i cst[MX_VECS];
    __shared__ v4i digits[8][MX_MAX_L * 2 * 64];
    __shared__ uint32_t accs[8][2 * MXN];
    for (int t = threadIdx.x; t < MX_VECS; t += 512) cst[t] = reinterpret_cast<const v4i *>(A.mx.cst)[t];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = (lane & 31) + 128 * (lane >> 5);  // + mx_off(v): the coefficient of register v
    uint32_t *const own = accs[wave] + base;
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
        uint32_t *const mine = accs[wave] + pos;
        // Phi(b') (0, V) or the stored state; each lane writes the words it alone reads back
        // as its own, and the step's first barrier makes them visible to the rotations
        if (has && (T.flags & TASK_INIT)) {
            uint32_t src, e;
            phi_row(__builtin_amdgcn_readfirstlane(modswitch_dev(ct[A.n], T.q_in, M)), r, T.comp, src, e);
            const uint32_t *V = A.tv + T.tv_off + (size_t)src * MXN;
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const uint32_t i2 = (pos + mx_off(v) + 2 * MXN - (e % (2 * MXN))) % (2 * MXN);
                const uint32_t x = V[i2 & (MXN - 1)];
                mine[mx_off(v)] = 0;
                mine[MXN + mx_off(v)] = (i2 >= (uint32_t)MXN) ? (x ? Q - x : 0) : x;
            }
        } else if (has) {
            const uint32_t *S = A.acc_state + T.acc_off + (size_t)T.comp * 2 * MXN + pos;
#pragma unroll
            for (int v = 0; v < 16; v++) {
                mine[mx_off(v)] = S[mx_off(v)];
                mine[MXN + mx_off(v)] = S[MXN + mx_off(v)];
            }
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
                    const uint32_t *sp = accs[wave - T.comp + src];
                    const uint32_t rb = (uint32_t)base + 2 * MXN - (e % (2 * MXN));
                    uint32_t y[2][16];
#pragma unroll
                    for (int v = 0; v < 16; v++) {
                        const uint32_t i2 = rb + mx_off(v);
                        const uint32_t at = i2 & (MXN - 1);
                        const uint32_t flip = 0u - ((i2 >> 10) & 1u);
                        const uint32_t fq = flip & (Q + 1);
                        y[0][v] = mx_field(sp[at], own[mx_off(v)], flip, fq, Q, A.mx, A.sg);
                        y[1][v] = mx_field(sp[MXN + at], own[MXN + mx_off(v)], flip, fq, Q, A.mx, A.sg);
                    }
                    mx_digits(y, A.l, A.log2B, A.mx, lane, dig);
                    mx_products(dig, cst, A.mx.bsk + ((size_t)i * KEYS + key) * (4u * A.l * MXN), A.l, lane, A.mx, m,
                                acc);
                    if (KEYS == 2 && key == 0) mx_fold(acc, A.mx);
                }
            }
            __syncthreads();  // every rotation of the step has read the accumulators
            if (active)
                mx_inverse(acc, cst, lane, A.mx, m, [&](int p, int v, uint32_t x) {
                    uint32_t *o = own + p * MXN + mx_off(v);
                    *o = add_q(*o, x, Q);
                });
        }
        if (has) {
            if (T.flags & TASK_STORE) {
                uint32_t *S = A.acc_state + T.acc_off + (size_t)T.comp * 2 * MXN + pos;
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    S[mx_off(v)] = mine[mx_off(v)];
                    S[MXN + mx_off(v)] = mine[MXN + mx_off(v)];
                }
            }
            if ((T.flags & TASK_EXTRACT) && T.comp == 0 && T.i0 + lim >= A.n) {
                // (A_0, -A_{N-1}, ..., -A_1; B_0) (eq. equ-sam-extr)
                uint32_t *o = A.ext_out + (size_t)T.ct * (MXN + 1);
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const uint32_t idx = pos + mx_off(v), x = mine[mx_off(v)];
                    o[(MXN - idx) & (MXN - 1)] = idx ? (x ? Q - x : 0) : x;
                }
                if (lane == 0) o[MXN] = mine[MXN];
            }
        }
        __syncthreads();  // the next group's accumulators take this one's place
    }
}

// ------------------------------------------------------------------ one CMux step

template <int KEYS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mx_step(WideArgs A, uint32_t num_tasks)
{
    __shared__ v4i cst[MX_VECS];
    __shared__ v4i digits[8][MX_MAX_L * 2 * 64];
    for (int t = threadIdx.x; t < MX_VECS; t += 512) cst[t] = reinterpret_cast<const v4i *>(A.mx.cst)[t];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int base = (lane & 31) + 128 * (lane >> 5);
    v4i *const dig = digits[wave];
    const uint32_t Q = A.Q[0];
    const ModS m{(int32_t)Q, A.qn[0]};
    const uint32_t slot = xcd_item(blockIdx.x, gridDim.x) * 8 + wave;
    for (uint32_t item = slot; item < num_tasks; item += gridDim.x * 8) {
        const WideTask &T = A.tasks[item];
        const uint32_t i = __builtin_amdgcn_readfirstlane(T.i0) + A.step;
        const uint32_t r = __builtin_amdgcn_readfirstlane(T.r), comp = __builtin_amdgcn_readfirstlane(T.comp);
        const uint32_t q_in = __builtin_amdgcn_readfirstlane(T.q_in);
        const uint64_t off = T.acc_off;
        const uint32_t *own = A.acc_rd + off + (size_t)comp * 2 * MXN + base;
        uint32_t *wr = A.acc_wr + off + (size_t)comp * 2 * MXN + base;
        if (i >= A.n) {
#pragma unroll
            for (int v = 0; v < 16; v++) {
                wr[mx_off(v)] = own[mx_off(v)];
                wr[MXN + mx_off(v)] = own[MXN + mx_off(v)];
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
            const uint32_t *sp = A.acc_rd + off + (size_t)src * 2 * MXN;
            const uint32_t rb = (uint32_t)base + 2 * MXN - (e % (2 * MXN));
            uint32_t y[2][16];
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const uint32_t i2 = rb + mx_off(v);
                const uint32_t at = i2 & (MXN - 1);
                const uint32_t flip = 0u - ((i2 >> 10) & 1u);
                const uint32_t fq = flip & (Q + 1);
                y[0][v] = mx_field(sp[at], own[mx_off(v)], flip, fq, Q, A.mx, A.sg);
                y[1][v] = mx_field(sp[MXN + at], own[MXN + mx_off(v)], flip, fq, Q, A.mx, A.sg);
            }
            mx_digits(y, A.l, A.log2B, A.mx, lane, dig);
            mx_products(dig, cst, A.mx.bsk + ((size_t)i * KEYS + key) * (4u * A.l * MXN), A.l, lane, A.mx, m, acc);
            if (KEYS == 2 && key == 0) mx_fold(acc, A.mx);
        }
        uint32_t old[2][16];  // this component's accumulator again, requested early
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int p = 0; p < 2; p++)
#pragma unroll
            for (int v = 0; v < 16; v++) old[p][v] = own[p * MXN + mx_off(v)];
        __builtin_amdgcn_sched_barrier(0);
        mx_inverse(acc, cst, lane, A.mx, m,
                   [&](int p, int v, uint32_t x) { wr[p * MXN + mx_off(v)] = add_q(old[p][v], x, Q); });
    }
}

// The bootstrapping key in this kernel's order: dst[poly][q][lane][s], entry of
// NTT position k = k1 + 32 k2 (k1 = lane % 32, k2 = 8 q + 4 (lane / 32) + s), from the
// bit-reversed, Montgomery-form key, times another 2^32 and balanced.
__global__ __launch_bounds__(256) void k_mx_keys(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                 uint32_t Q, uint32_t qn, uint32_t two64)
{
    constexpr int N = MXN;
    const size_t base = (size_t)blockIdx.x * N;
    const ModQ m{Q, qn};
    for (int t = threadIdx.x; t < N; t += 256) {
        const int q = t >> 8, lane = (t >> 2) & 63, s = t & 3;
        const uint32_t k = (lane & 31) + 32 * (8 * q + 4 * (lane >> 5) + s);
        const uint32_t x = mont_mul(src[base + (__brev(k) >> 22)], two64, m);
        dst[base + t] = x > (Q - 1) / 2 ? x - Q : x;
    }
}

void launch_mx_keys(const uint32_t *src, uint32_t *dst, size_t polys, uint32_t Q, uint32_t qn, uint32_t two64,
                    hipStream_t st)
{
    hipLaunchKernelGGL(k_mx_keys, dim3((uint32_t)polys), dim3(256), 0, st, src, dst, Q, qn, two64);
}

void launch_mx_rotate(const BrArgs &A, int grid, hipStream_t st)
{
    if (A.keys == 2) hipLaunchKernelGGL(k_mx_rotate<2>, dim3(grid), dim3(512), 0, st, A);
    else hipLaunchKernelGGL(k_mx_rotate<1>, dim3(grid), dim3(512), 0, st, A);
}

void launch_mx_step(uint32_t keys, const WideArgs &A, uint32_t num_tasks, hipStream_t st)
{
    const uint32_t grid = std::min<uint32_t>((num_tasks + 7) / 8, A.mx.num_cu);
    if (keys == 2) hipLaunchKernelGGL(k_mx_step<2>, dim3(grid), dim3(512), 0, st, A, num_tasks);
    else hipLaunchKernelGGL(k_mx_step<1>, dim3(grid), dim3(512), 0, st, A, num_tasks);
}

}  // namespace dev
}  // namespace mm
