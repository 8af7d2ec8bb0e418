// The half-sweep of one 16-byte run, shared by the kernels that keep several half-sweeps on the chip.
#pragma once
#include "mg_internal.h"
#include "p2_bodies.h"

namespace mgic {

template <class T>
using V16 = typename Vec16<T>::type;

template <class T>
__device__ __forceinline__ V16<T> pack(const T* v) {
    if constexpr (Vec16<T>::W == 4) return V16<T>{v[0], v[1], v[2], v[3]};
    else return V16<T>{v[0], v[1]};
}

// one run of a half-sweep: x-neighbours xm, xp, y-neighbours ym, yp, the other colour's run c of the own
// row with the neighbouring entry `edge` (after it for q = 1, before it for q = 0), right-hand side f
template <class T>
__device__ __forceinline__ V16<T> update_run(const V16<T>& xm, const V16<T>& xp, const V16<T>& ym, const V16<T>& yp,
                                             const V16<T>& c, T edge, const V16<T>& f, bool q, T h2) {
    constexpr int W = Vec16<T>::W;
    T out[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const T before = k == 0 ? edge : lane<T>(c, k - 1), after = k == W - 1 ? edge : lane<T>(c, k + 1);
        const T z = (q ? after : before) + lane<T>(c, k);
        const T s = ((lane<T>(xm, k) + lane<T>(xp, k)) + (lane<T>(ym, k) + lane<T>(yp, k))) + z;
        out[k] = div6(s - h2 * lane<T>(f, k));
    }
    return pack<T>(out);
}

}  // namespace mgic
