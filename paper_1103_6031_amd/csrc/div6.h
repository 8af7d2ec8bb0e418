// x / c for a constant c, rounded to nearest by a multiplication and two fused multiply-adds: with
// r = RN(1/c) and q = RN(x r), the remainder x - c q is exact and RN(q + r (x - c q)) is the correctly rounded
// quotient (P. Markstein, "Computation of elementary functions on the IBM RISC System/6000 processor",
// IBM J. Res. Dev. 34, 1990, theorem on a correctly rounded reciprocal) wherever the remainder
// is no denormal number: for c = 6 wherever the quotient is none, for any constant from |q| = 2^-104 (FP32) and
// 2^-971 (FP64) on; below, the last place may be off.  Zeros, infinities and NaN are those of the division.
// The compiler's division takes about ten instructions.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define MGIC_DIV6_HD __host__ __device__ __forceinline__
#else
#define MGIC_DIV6_HD inline
#endif

namespace mgic {

MGIC_DIV6_HD float div_const(float x, float c) {
    const float r = 1.0f / c;
    float q = x * r;
    q = fmaf(fmaf(-c, q, x), r, q);
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_div_fixupf(q, c, x);
#else
    return std::isfinite(x) && x != 0.0f ? q : x * (c < 0.0f ? -1.0f : 1.0f);
#endif
}

MGIC_DIV6_HD double div_const(double x, double c) {
    const double r = 1.0 / c;
    double q = x * r;
    q = fma(fma(-c, q, x), r, q);
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_div_fixup(q, c, x);
#else
    return std::isfinite(x) && x != 0.0 ? q : x * (c < 0.0 ? -1.0 : 1.0);
#endif
}

MGIC_DIV6_HD float div6(float x) { return div_const(x, 6.0f); }
MGIC_DIV6_HD double div6(double x) { return div_const(x, 6.0); }

}  // namespace mgic
