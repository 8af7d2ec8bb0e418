// x / 6 rounded to nearest by a multiplication and two fused multiply-adds: with r = RN(1/6) and
// q = RN(x r), the remainder x - 6 q is exact and RN(q + r (x - 6 q)) is the correctly rounded
// quotient (P. Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor",
// IBM J. Res. Dev. 34, 1990, theorem on a correctly rounded reciprocal) wherever it is a normal number;
// a denormal one may be off by its last place.  Zeros, infinities and NaN are those of the division.
// The compiler's division takes about ten instructions.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#define MGIC_DIV6_HD __host__ __device__ __forceinline__
#else
#define MGIC_DIV6_HD inline
#endif

namespace mgic {

MGIC_DIV6_HD float div6(float x) {
    const float r = 1.0f / 6.0f;
    float q = x * r;
    q = fmaf(fmaf(-6.0f, q, x), r, q);
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_div_fixupf(q, 6.0f, x);
#else
    return std::isfinite(x) && x != 0.0f ? q : x;
#endif
}

MGIC_DIV6_HD double div6(double x) {
    const double r = 1.0 / 6.0;
    double q = x * r;
    q = fma(fma(-6.0, q, x), r, q);
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_div_fixup(q, 6.0, x);
#else
    return std::isfinite(x) && x != 0.0 ? q : x;
#endif
}

}  // namespace mgic
