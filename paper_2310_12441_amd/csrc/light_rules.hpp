// Which shape takes light work at N = 1024, and work of two primes at N = 2048: one rule for
// batches and for a server's ticks.
#pragma once

#include <cstdint>

namespace mm {

struct LightWork {
    uint64_t comps;  // ring components in all
    uint32_t max_r;  // of the widest ciphertext
    uint32_t keys;   // RGSW keys per coordinate (2: ternary secret)
    uint64_t cu;     // compute units
    bool mx;         // the matrix-core kernels of one prime apply
    bool beside = false;  // a fused kernel of other work runs at the same time (a server's other partition)
};

// The matrix-core kernel with two waves per component (630 steps, ms): up to four components
// per compute unit where every ciphertext fits such slots (148 components 7.0, 400 7.9, 1024 9.2;
// two digit groups 7.5, 11.0, 19.1; one wave 8.0, 8.8, 9.6; with r <= 2 from the first ciphertext
// on, 4.2 against 6.1 for one of r = 1; with r = 4 one takes 6.3 either way and up to 16
// components keep the digit groups; with a ternary secret up to 48, whole calls of r = 4: 20
// components 10.8 against 11.1, 64 11.15 either way).  The lines at 16 and 48 are where a single
// ciphertext's chain of steps, not the compute units, sets the time: they do not grow with the device.
inline bool two_mx_waves(const LightWork &w)
{
    return w.mx && w.max_r <= 4 && w.comps <= 4 * w.cu && (w.max_r <= 2 || w.comps > (w.keys == 2 ? 48u : 16u));
}

// One launch per step, four waves per component: where the matrix-core kernels apply up to two
// components per compute unit (r = 8, ms: 264 components 9.5 against 11.2 with one wave per
// component, 512 9.9 against 11.2, 640 13.9 against 11.3; ternary 264 16.0 against 19.9, 512 16.4
// against 20.0, 640 23.4 against 19.9), beside a fused kernel, whose workgroups hold their compute units for a
// whole tick, up to one (16,000 requests/s of r = 1, 2, 4, 8, p50 of those of r = 8: 14.6 ms, 16.2 with up to
// two; 10,000 11.3 and 10.8); without them the batches that leave the device mostly idle:
// two components per compute unit, or four where the components cannot take two-wave slots (one
// ciphertext 7.4 ms instead of 14.2 ms, or 25.9 ms at r = 8).
inline bool steps_by_launch(const LightWork &w)
{
    if (w.mx) return !two_mx_waves(w) && w.comps <= (w.beside ? 1 : 2) * w.cu;
    return w.comps <= 2 * w.cu || (w.max_r > 4 && w.comps <= 4 * w.cu);
}

// Two primes at N = 2048 beside the matrix-core kernels: one matrix-core workgroup per component
// and prime (6), the butterfly workgroup per component and prime (5), or the matrix-core step of two
// components per workgroup (0).  5 and 6 take time by rounds of one component for every two
// compute units, 0 by rounds of four times as many.  The matrix cores work on pairs of digits, an
// odd length with a zero polynomial behind it, so they gain least at l = 1 and, with one key, at
// l = 2 and 3.  100 steps, ms, one key unless said (components: 6 / 5 / 0):
//   l = 1  128: 1.33 / 1.32 / 2.77, 384: 3.29 / 2.15 / 3.22, 1024: - / 4.86 / 5.71; two keys 384:
//          4.02 / 3.10 / 4.03, 1024: - / 7.34 / 7.63
//   l = 2  128: 1.35 / 1.61 / 2.75, 384: 3.29 / 2.77 / 3.18, 512: - / 3.55 / 3.39, 768: - / 4.97 / 5.59, 1024: -
//          / 6.38 / 5.82; two keys 384: 4.12 / 4.39 / 4.06, 768: - / 8.08 / 7.74
//   l = 3  128: 1.51 / 1.90 / 3.47, 384: 3.73 / 3.37 / 3.96, 512: - / 4.38 / 4.24, 768: - / 6.12 / 7.17, 1024: -
//          / 7.89 / 7.41; two keys 384: 5.31 / 5.66 / 5.40
//   l = 4  384: 3.77 / 4.00 / 3.91, 768: - / 7.29 / 7.28; two keys 384: 5.43 / 6.90 / 5.45, 768: - / 12.8 / 11.3
inline int two_prime_shape(uint64_t comps, uint32_t l, uint32_t keys, uint64_t cu)
{
    const uint64_t rounds = (2 * comps + cu - 1) / cu;
    if (rounds <= 1) return 6;
    if (l == 1) return 5;
    const bool lean = keys == 1 && l <= 3;
    if (rounds <= 3) return lean ? 5 : 6;
    const uint64_t last = (rounds - 1) % 4 + 1;  // of the step's last round, quarters
    return lean && rounds <= 14 && last <= 2 ? 5 : 0;
}

}  // namespace mm
