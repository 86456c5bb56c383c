// The correctly rounded binary32 root from one that is off by at most one unit; host and device.
#ifndef ISR_NEAREST_ROOT_H
#define ISR_NEAREST_ROOT_H

#include <hip/hip_runtime.h>

namespace isr {

__host__ __device__ inline float float_next(float f, int units) {
    union { float f; uint32_t u; } b = {f};
    b.u += (uint32_t)units;
    return b.f;
}

// The root of x >= 0 (0, or far from the ends of the range) from s, at most one unit u away.  It lies below the middle of s - u and s
// where x < (s - u/2)^2 = s (s - u) + u^2/4; x - s (s - u) is a multiple of u^2, so that is where it is not positive, and one fused
// multiply-add has its sign.  The same above s.  This is the usual correction by the residuals at the neighbours (compilers expand
// a correctly rounded root this way).  tests/test_nearest_root_host.py goes through all mantissas of both parities of the exponent.
__host__ __device__ inline float nearest_root(float x, float s) {
    const float below = float_next(s, -1), above = float_next(s, 1);   // of 0: NaN, which is neither
    const float r = __builtin_fmaf(-below, s, x) <= 0.0f ? below : s;
    return __builtin_fmaf(-above, s, x) > 0.0f ? above : r;
}

}  // namespace isr

#endif
