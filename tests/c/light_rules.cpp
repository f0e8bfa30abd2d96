// Prints the shape that light_rules.hpp gives light work: one line per
// "comps max_r keys cu mx beside" read.
#include <cstdio>

#include "light_rules.hpp"

int main()
{
    unsigned long long comps, cu;
    unsigned max_r, keys, mx, beside;
    while (std::scanf("%llu %u %u %llu %u %u", &comps, &max_r, &keys, &cu, &mx, &beside) == 6) {
        const mm::LightWork w{comps, max_r, keys, cu, mx != 0, beside != 0};
        std::puts(mm::two_mx_waves(w) ? "two waves" : mm::steps_by_launch(w) ? "steps" : "one wave");
    }
}
