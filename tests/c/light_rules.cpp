// Prints the shape that light_rules.hpp gives work: one line per "comps max_r keys cu mx beside" read,
// or, with an argument, per "comps l keys cu" of two primes.
#include <cstdio>

#include "light_rules.hpp"

int main(int argc, char **)
{
    unsigned long long comps, cu;
    unsigned max_r, keys, mx, beside;
    while (argc > 1 && std::scanf("%llu %u %u %llu", &comps, &max_r, &keys, &cu) == 4)
        std::printf("%d\n", mm::two_prime_shape(comps, max_r, keys, cu));
    while (std::scanf("%llu %u %u %llu %u %u", &comps, &max_r, &keys, &cu, &mx, &beside) == 6) {
        const mm::LightWork w{comps, max_r, keys, cu, mx != 0, beside != 0};
        std::puts(mm::two_mx_waves(w) ? "two waves" : mm::steps_by_launch(w) ? "steps" : "one wave");
    }
}
