// Host check of mgic::div_const, for the divisors of the higher-order smoothers (three times the central
// weight of orders 2, 4 and 6), against the hardware division (built with g++ -mfma by
// tests/test_native_div6.py).  The remainder x - c q is a multiple of ulp(c) ulp(q), 2^-21 2^-23 |q| in FP32
// and 2^-50 2^-52 |q| in FP64 for 4 <= |c| < 16, so it is exact, and the quotient the correctly rounded one,
// while that is no denormal: from |q| = 2^-104 and 2^-971 on.  Below, the last place may differ.
#include <cstdint>
#include <cstdio>
#include <cstring>

#include "div6.h"

template <class T, class U>
static bool agrees(U bits, T c, T smallest) {
    T x;
    memcpy(&x, &bits, sizeof x);
    const T a = mgic::div_const(x, c), b = x / c;
    if (x != x) return a != a;
    if (x != T(0) && (b < T(0) ? -b : b) < smallest) {
        U ua, ub;
        memcpy(&ua, &a, sizeof a);
        memcpy(&ub, &b, sizeof b);
        return ua - ub + 1 <= 2;                                     // neighbours at most
    }
    return memcmp(&a, &b, sizeof a) == 0;
}

int main() {
    unsigned long long bad = 0, s = 88172645463325252ull;
    const double w0[3] = {-2.0, -30.0 / 12, -490.0 / 180};
    for (double w : w0) {
        const float cf = 3.0f * (float)w;
        const double cd = 3.0 * w;
        for (uint32_t m = 0; m < (1u << 23); ++m) bad += !agrees<float>(0x3f800000u | m, cf, 0x1p-104f);
        for (uint32_t e = 0; e < 512; ++e)
            for (uint32_t m = 0; m < (1u << 23); m += 4099) bad += !agrees<float>((e << 23) | m, cf, 0x1p-104f);
        for (int i = 0; i < 10000000; ++i) {
            s ^= s << 13; s ^= s >> 7; s ^= s << 17;
            bad += !agrees<double>((uint64_t)s, cd, 0x1p-971);
        }
    }
    printf("mismatches %llu\n", bad);
    return bad ? 1 : 0;
}
