// The reductions that end in balanced bytes (mx_twist and mx_cut of kernels_mx.hip), a value at a
// time, with their wrapping multiply-adds, against exact 128-bit arithmetic.  Built with
// checks of signed overflow.  Usage: wrap64 Q
#include <cstdio>
#include <cstdlib>
#include <random>

#include "wrap64.hpp"

using mm::dev::mad_wrap;

int main(int argc, char **argv)
{
    if (argc != 2) return 2;
    const uint32_t Q = (uint32_t)std::strtoul(argv[1], nullptr, 10), BAL = 0x80808080u;
    uint32_t inv = 1;  // Q^-1 mod 2^32
    for (int k = 0; k < 5; k++) inv *= 2u - Q * inv;
    const int64_t bal64 = (int64_t)((uint64_t)BAL << 32);
    const int32_t half = (int32_t)(Q / 2);
    std::mt19937 rng(Q);
    auto pick = [&](int32_t most) {  // the ends of [-most, most] and values between
        const int32_t v = (int32_t)((int64_t)(rng() % (2ull * (uint32_t)most + 1)) - most);
        return rng() % 4 ? v : v < 0 ? -most : most;
    };
    long bad = 0;
    auto check = [&](int64_t t, __int128 exact) {
        const int32_t q = (int32_t)((uint32_t)t * (0u - inv));
        const int32_t o = (int32_t)(mad_wrap(q, (int32_t)Q, t) >> 32);
        const uint32_t z = (uint32_t)o ^ BAL;
        int64_t x = 0;
        for (int j = 0; j < 4; j++) x += (int64_t)(int8_t)(z >> (8 * j)) << (8 * j);
        const __int128 m = (__int128)x * ((__int128)1 << 32) - exact;
        bad += m % Q != 0 || x > (1ll << 31) - 1 - 0x808080 || x < -(1ll << 31);
    };
    const int32_t join = 1 << 30, two32 = (int32_t)(((uint64_t)1 << 32) % Q);
    const int32_t two32c = two32 > half ? (int32_t)((uint32_t)two32 - Q) : two32;
    for (int k = 0; k < 2000000; k++) {
        const int32_t hi = pick(join), lo = pick(join), w = pick(half), w16 = pick(half);
        check(mad_wrap(lo, w, mad_wrap(hi, w16, bal64)), (__int128)hi * w16 + (__int128)lo * w);
        const int32_t high = pick(0x7fffffff);
        const uint32_t low = rng();
        check(mad_wrap(high, two32c, (int64_t)(low | (uint64_t)BAL << 32)), (__int128)high * two32c + low);
    }
    std::printf("%ld wrong\n", bad);
    return bad != 0;
}
