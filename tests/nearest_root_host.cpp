// nearest_root for every binary32 x in [1, 4) -- all mantissas, both parities of the exponent; a factor of 4 changes nothing -- from the
// correctly rounded root and from one unit to either side, at the scales of the sampler's smallest, middle and largest arguments, and 0.
// Against the binary64 root, whose rounding to binary32 is the correct one (it has more than twice the digits and two).
// Built and run by tests/test_nearest_root_host.py.
#include <cmath>
#include <cstdint>
#include <cstdio>

#include "nearest_root.h"

int main() {
    long checked = 0;
    for (int scale : {-24, 0, 4})   // x from 2^-24 to 64
        for (uint32_t u = 0; u < 1u << 24; ++u) {
            const float x = std::ldexp(isr::float_next(1.0f, (int)u), scale);
            const float want = (float)std::sqrt((double)x);
            for (int off : {-1, 0, 1}) {
                const float got = isr::nearest_root(x, isr::float_next(want, off));
                ++checked;
                if (got != want) {
                    std::printf("x %a from %+d: %a instead of %a\n", x, off, got, want);
                    return 1;
                }
            }
        }
    if (isr::nearest_root(0.0f, 0.0f) != 0.0f) return 1;
    std::printf("checked %ld\n", checked);
    return 0;
}
