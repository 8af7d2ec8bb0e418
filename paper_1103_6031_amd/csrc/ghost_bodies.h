// The covered parent cell of a level's cell, and the parts of a patch's ghost values.
#pragma once
#include "mg_internal.h"

namespace mgic {

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

// index of covered cell (X,Y,Z) (relative to the covered box) in the parent array
__device__ __forceinline__ size_t pidx(const ParentMap& pm, int X, int Y, int Z) {
    int a = pm.off[0] + X, b = pm.off[1] + Y, c = pm.off[2] + Z;
    if (pm.periodic) {
        a = wrap(a, pm.pl.d.x);
        b = wrap(b, pm.pl.d.y);
        c = wrap(c, pm.pl.d.z);
    }
    return lidx(pm.pl.d, pm.pl.split, a, b, c);
}

// ----------------------------------------------------------------------------------------------
// coarse-fine ghost zones with flux matching (Section 3.3, Table 2 order-1 flux), computed per 2x2
// group of fine face cells sharing a parent C.  For the low-x face and fine cell (0, j, k):
//   a  = quadratic interpolation in the outside parent layer at the child's transverse position
//   g0 = 8/15 a + 2/3 u0 - 1/5 u1            (quadratic normal to the face)
//   g  = g0 + (mean u0 - mean g0) - 1/2 (mean8(children of C) - U[O])
// so the mean fine flux (u0 - g)/h through the coarse face equals the coarse flux (C - O)/(2h),
// with C taken as the live mean of its children.  Other faces mirror this.
// ----------------------------------------------------------------------------------------------

__device__ __forceinline__ void w2(double t, double w[3]) {
    w[0] = 0.5 * t * (t - 1.0);
    w[1] = 1.0 - t * t;
    w[2] = 0.5 * t * (t + 1.0);
}

// component k of a triple (selects: an index known at run time only would put the array in scratch memory)
__device__ __forceinline__ int pick(int k, int x, int y, int z) { return k == 0 ? x : (k == 1 ? y : z); }
// 3 x 3 cells of the outside parent layer around the parent cell O in front of group (J, K) of a face
template <class T>
__device__ __forceinline__ void ghost_parent(const T* __restrict__ pu, const ParentMap& pm, const Dims& d, int face,
                                             int J, int K, double L[3][3]) {
    const int a = face >> 1, side = face & 1;
    const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;
    const int oa = pick(a, pm.off[0], pm.off[1], pm.off[2]);
    const int on = side ? oa + pick(a, d.x, d.y, d.z) / 2 : oa - 1;
    const int ob = pick(b, pm.off[0], pm.off[1], pm.off[2]) + J - 1, oc = pick(c, pm.off[0], pm.off[1], pm.off[2]) + K - 1;
#pragma unroll
    for (int db = 0; db < 3; ++db)
#pragma unroll
        for (int dc = 0; dc < 3; ++dc) {
            int x = a == 0 ? on : ob + db, y = a == 1 ? on : (a == 0 ? ob + db : oc + dc), z = a == 2 ? on : oc + dc;
            if (pm.periodic) {
                x = wrap(x, pm.pl.d.x);
                y = wrap(y, pm.pl.d.y);
                z = wrap(z, pm.pl.d.z);
            }
            L[db][dc] = (double)pu[lidx(pm.pl.d, pm.pl.split, x, y, z)];
        }
}
// their interpolation at child (jb, kc): parallel to the face, first along b (for each of the 3
// c-columns), then along c
__device__ __forceinline__ double ghost_interp(const double L[3][3], int jb, int kc) {
    double wb[3], wc[3];
    w2(jb ? 0.25 : -0.25, wb);
    w2(kc ? 0.25 : -0.25, wc);
    double Ab[3];
#pragma unroll
    for (int dc = 0; dc < 3; ++dc) Ab[dc] = (wb[0] * L[0][dc] + wb[1] * L[1][dc]) + wb[2] * L[2][dc];
    return (wc[0] * Ab[0] + wc[1] * Ab[1]) + wc[2] * Ab[2];
}
__device__ __forceinline__ double ghost_g0(double aq, double u0, double u1) {
    return ((8.0 / 15.0) * aq + (2.0 / 3.0) * u0) - 0.2 * u1;
}
__device__ __forceinline__ double ghost_shift(double m_u0, double m_u1, double m_g0, double O) {
    const double uC = 0.5 * (m_u0 + m_u1);
    return (m_u0 - m_g0) - 0.5 * (uC - O);
}

}  // namespace mgic
