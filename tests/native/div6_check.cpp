// Host check of mgic::div6 against the hardware division (built with g++ -mfma by tests/test_native_div6.py).
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <initializer_list>
#include "div6.h"

template <class T, class U>
static bool agrees(U bits, T smallest) {
    T x;
    memcpy(&x, &bits, sizeof x);
    if (x != x) return mgic::div6(x) != mgic::div6(x);
    const T a = mgic::div6(x), b = x / T(6);
    if (x != T(0) && (b < T(0) ? -b : b) < smallest) return true;   // a denormal quotient
    return memcmp(&a, &b, sizeof a) == 0;
}

int main() {
    unsigned long long bad = 0, s = 88172645463325252ull;
    // every mantissa of one FP32 binade of each sign, every exponent with some mantissas, FP64 at random
    for (uint32_t m = 0; m < (1u << 23); ++m)
        for (uint32_t e : {0x3f800000u, 0xc0000000u}) bad += !agrees<float>(e | m, 0x1p-126f);
    for (uint32_t e = 0; e < 512; ++e)
        for (uint32_t m = 0; m < (1u << 23); m += 997) bad += !agrees<float>((e << 23) | m, 0x1p-126f);
    for (int i = 0; i < 20000000; ++i) {
        s ^= s << 13; s ^= s >> 7; s ^= s << 17;
        bad += !agrees<double>((uint64_t)s, 0x1p-1022);
    }
    printf("mismatches %llu\n", bad);
    return bad ? 1 : 0;
}
