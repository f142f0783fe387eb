// hmf_terms.h -- per-particle helpers of the HMF kernels (hmf.hip, hmf_small.hip).
#pragma once

#include "device.h"

namespace md {

// sincos of E angles, each step over all of them before the next, so that their
// chains interleave.  FP64: the branch-free reduced form for all, then the library
// for any angle beyond its range (never, for the dynamics here).
template <int E>
__device__ __forceinline__ void sincos_n(const double (&x)[E], double (&s)[E], double (&c)[E])
{
    bool big = false;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        sincos64_reduced(x[e], &s[e], &c[e]);
        big |= !(fabs(x[e]) < kSincosMaxArg);
    }
    if (big) {
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (!(fabs(x[e]) < kSincosMaxArg)) sincos(x[e], &s[e], &c[e]);
    }
}
template <int E>
__device__ __forceinline__ void sincos_n(const float (&x)[E], float (&s)[E], float (&c)[E])
{
#pragma unroll
    for (int e = 0; e < E; ++e) sincos32(x[e], &s[e], &c[e]);
}

// Map an FP32 angle into [-pi, pi).
__device__ __forceinline__ float wrap_pi(float t)
{
    const float two_pi = 6.28318530717958647692f;
    const float k = rintf(t * 0.159154943091895335769f);
    t = __builtin_fmaf(-k, two_pi, t);
    if (t >= 3.14159265358979323846f) t -= two_pi;
    if (t < -3.14159265358979323846f) t += two_pi;
    return t;
}

}  // namespace md
