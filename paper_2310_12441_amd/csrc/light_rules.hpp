// Which shape takes light work at N = 1024: one rule for batches and for a server's ticks.
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

}  // namespace mm
