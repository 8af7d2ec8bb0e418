// LPT kernels for gfx950 (Hahn & Abel 2011, Section 3.1, and the baryon density of Section 5.3):
//   first order   psi_c = scale * G_c phi            (Table 1 gradient, fourth or sixth order)
//   second order  tau = sum_{i>j} D_ii D_jj - D_ij^2,  D_ij = G_i (G_j phi)
//   LLA density   rho / rho_bar - 1 = 1 / det(I + G4 L) - 1   (eq. gasdens)
// plus the post-solve ghost layers of width R (faces, edges and corners) that patches need:
// coarse-only tri-quadratic interpolation of the parent at the child's position (children sit at
// -1/4 and +1/4 of the parent cell along each axis).
//
// Sources are either periodic n^3 arrays (indices wrap) or arrays padded by R ghost cells on
// every side; the two cases are separate instantiations.  The gradient is evaluated as
// ((u[-2] - 8 u[-1]) + 8 u[+1]) - u[+2], / (12 h), then scaled.  tau takes two passes:
// psi_j = G4_j phi is stored (extended by 2 cells on patches), then D_ij = G4_i psi_j is
// evaluated per cell.  Output cells are decoded from a linear index with multiply-shift
// division (every array has fewer than 2^31 cells).  Periodic levels take groups of rows, and
// where the tile divides the level, x-marched tiles with a ring of plane slabs in LDS.

#include <initializer_list>

#include "mg_internal.h"

namespace mgic {

template <bool PAD>
struct Src {
    const double* p;
    int R;    // padding (PAD) - unused when periodic
    Dims d;   // interior dims
    __device__ __forceinline__ double at(int x, int y, int z) const {
        if constexpr (!PAD) {
            x = x < 0 ? x + d.x : (x >= d.x ? x - d.x : x);
            y = y < 0 ? y + d.y : (y >= d.y ? y - d.y : y);
            z = z < 0 ? z + d.z : (z >= d.z ? z - d.z : z);
            return p[((unsigned)x * d.y + y) * (unsigned)d.z + z];
        } else {
            const unsigned py = (unsigned)d.y + 2 * R, pz = (unsigned)d.z + 2 * R;
            return p[((unsigned)(x + R) * py + (y + R)) * pz + (z + R)];
        }
    }
};

// fourth-order gradient of s along `axis` at (x, y, z), Table 1 weights (1, -8, 0, 8, -1) / 12
template <bool PAD>
__device__ __forceinline__ double g4(const Src<PAD>& s, int x, int y, int z, int axis, double den) {
    const int ex = axis == 0, ey = axis == 1, ez = axis == 2;
    double acc = s.at(x - 2 * ex, y - 2 * ey, z - 2 * ez);
    acc = acc + (-8.0) * s.at(x - ex, y - ey, z - ez);
    acc = acc + 8.0 * s.at(x + ex, y + ey, z + ez);
    acc = acc + (-1.0) * s.at(x + 2 * ex, y + 2 * ey, z + 2 * ez);
    return acc / den;
}

// sixth-order gradient of s along `axis`, Table 1 weights (-1, 9, -45, 0, 45, -9, 1) / 60
template <bool PAD>
__device__ __forceinline__ double g6(const Src<PAD>& s, int x, int y, int z, int axis, double den) {
    const int ex = axis == 0, ey = axis == 1, ez = axis == 2;
    double acc = (-1.0) * s.at(x - 3 * ex, y - 3 * ey, z - 3 * ez);
    acc = acc + 9.0 * s.at(x - 2 * ex, y - 2 * ey, z - 2 * ez);
    acc = acc + (-45.0) * s.at(x - ex, y - ey, z - ez);
    acc = acc + 45.0 * s.at(x + ex, y + ey, z + ez);
    acc = acc + (-9.0) * s.at(x + 2 * ex, y + 2 * ey, z + 2 * ez);
    acc = acc + s.at(x + 3 * ex, y + 3 * ey, z + 3 * ez);
    return acc / den;
}

// the gradient of order G (4 or 6) with its denominator (12 h or 60 h)
template <bool PAD, int G>
__device__ __forceinline__ double gG(const Src<PAD>& s, int x, int y, int z, int axis, double h) {
    if constexpr (G == 4) return g4(s, x, y, z, axis, 12.0 * h);
    else return g6(s, x, y, z, axis, 60.0 * h);
}

// linear index -> (x, y, z) of a box, natural order
__device__ __forceinline__ void decode3(const Lay& B, unsigned t, int& x, int& y, int& z) {
    const unsigned row = B.dz.div(t);
    z = (int)(t - row * (unsigned)B.d.z);
    const unsigned xq = B.dy.div(row);
    y = (int)(row - xq * (unsigned)B.d.y);
    x = (int)xq;
}

template <bool PAD, int G = 4>
__global__ void k_grad4(Src<PAD> s, Lay B, double h, double scale, double* __restrict__ ox,
                        double* __restrict__ oy, double* __restrict__ oz) {
    const unsigned t = (unsigned)lpt_block() * blockDim.x + threadIdx.x;
    if (t >= (unsigned)B.d.cells()) return;
    int x, y, z;
    decode3(B, t, x, y, z);
    ox[t] = scale * gG<PAD, G>(s, x, y, z, 0, h);
    oy[t] = scale * gG<PAD, G>(s, x, y, z, 1, h);
    oz[t] = scale * gG<PAD, G>(s, x, y, z, 2, h);
}

// psi_j = G_j phi on the interior extended by e cells (e <= R - G / 2), unscaled; the output box
// B is (d + 2e)^3, padded by e
template <bool PAD, int G = 4>
__global__ void k_psi(Src<PAD> s, Lay B, int e, double h, double* __restrict__ p0, double* __restrict__ p1,
                      double* __restrict__ p2) {
    const unsigned t = (unsigned)lpt_block() * blockDim.x + threadIdx.x;
    if (t >= (unsigned)B.d.cells()) return;
    int x, y, z;
    decode3(B, t, x, y, z);
    x -= e;
    y -= e;
    z -= e;
    p0[t] = gG<PAD, G>(s, x, y, z, 0, h);
    p1[t] = gG<PAD, G>(s, x, y, z, 1, h);
    p2[t] = gG<PAD, G>(s, x, y, z, 2, h);
}

// tau = sum_{i>j} D_ii D_jj - D_ij^2 with D_ij = G_i psi_j; psi periodic or padded by e.  When
// psi is a scaled gradient s G phi, post = 1 / s^2 brings tau back to the one of phi (post = 1:
// not applied, so s = +-1 gives the same bits as psi = G phi)
template <bool PAD, int G = 4>
__global__ void k_tau_psi(Src<PAD> q0, Src<PAD> q1, Src<PAD> q2, Lay B, double h, double post,
                          double* __restrict__ tau) {
    const unsigned t = (unsigned)lpt_block() * blockDim.x + threadIdx.x;
    if (t >= (unsigned)B.d.cells()) return;
    int x, y, z;
    decode3(B, t, x, y, z);
    const double Dxx = gG<PAD, G>(q0, x, y, z, 0, h);
    const double Dyy = gG<PAD, G>(q1, x, y, z, 1, h);
    const double Dzz = gG<PAD, G>(q2, x, y, z, 2, h);
    const double Dyx = gG<PAD, G>(q0, x, y, z, 1, h);
    const double Dzx = gG<PAD, G>(q0, x, y, z, 2, h);
    const double Dzy = gG<PAD, G>(q1, x, y, z, 2, h);
    double acc = 0.0;
    acc = acc + (Dyy * Dxx - Dyx * Dyx);
    acc = acc + (Dzz * Dxx - Dzx * Dzx);
    acc = acc + (Dzz * Dyy - Dzy * Dzy);
    tau[t] = post == 1.0 ? acc : acc * post;
}

// LLA baryon density (Section 5.3, eq. gasdens): rho / rho_bar - 1 = 1 / det(I + J) - 1 with
// J_ij = G4_j L_i, where the displacement L is a (+ b when `sum`, formed per load, the same
// add a separate pass would make).  The stencil sums are multiplied by 1 / (12 h) (as g4m), and
// the determinant is expanded along the first row of M = I + J.
template <bool PAD>
__device__ __forceinline__ double g4_of(const Src<PAD>& a, const Src<PAD>& b, int sum, int x, int y, int z,
                                        int axis, double inv) {
    const int ex = axis == 0, ey = axis == 1, ez = axis == 2;
    auto v = [&](int k) {
        const int X = x + k * ex, Y = y + k * ey, Z = z + k * ez;
        return sum ? a.at(X, Y, Z) + b.at(X, Y, Z) : a.at(X, Y, Z);
    };
    double acc = v(-2);
    acc = acc + (-8.0) * v(-1);
    acc = acc + 8.0 * v(1);
    acc = acc + (-1.0) * v(2);
    return acc * inv;
}

template <bool PAD>
__global__ void k_lla(Src<PAD> a0, Src<PAD> a1, Src<PAD> a2, Src<PAD> b0, Src<PAD> b1, Src<PAD> b2, int sum,
                      Lay B, double h, double* __restrict__ out) {
    const unsigned t = (unsigned)lpt_block() * blockDim.x + threadIdx.x;
    if (t >= (unsigned)B.d.cells()) return;
    int x, y, z;
    decode3(B, t, x, y, z);
    const double inv = 1.0 / (12.0 * h);
    const Src<PAD>* A[3] = {&a0, &a1, &a2};
    const Src<PAD>* Bs[3] = {&b0, &b1, &b2};
    double m[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) m[i][j] = (i == j ? 1.0 : 0.0) + g4_of(*A[i], *Bs[i], sum, x, y, z, j, inv);
    const double c0 = m[1][1] * m[2][2] - m[1][2] * m[2][1];
    const double c1 = m[1][0] * m[2][2] - m[1][2] * m[2][0];
    const double c2 = m[1][0] * m[2][1] - m[1][1] * m[2][0];
    const double det = (m[0][0] * c0 - m[0][1] * c1) + m[0][2] * c2;
    out[t] = 1.0 / det - 1.0;
}

__global__ void k_add2(const double* __restrict__ a, const double* __restrict__ b, double* __restrict__ dst, size_t n) {
    for (size_t i = (size_t)lpt_block() * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = a[i] + b[i];
}

// ----------------------------------------------------------------------------------------------
// Periodic natural-order arrays, by groups of rows: one workgroup per (x, 8 consecutive y), each
// thread one z walking the 8 rows with the y-stencil values in a register window.  The blocks of
// one x plane are spread over the XCDs in turn, so with one block per row every row would be
// fetched into the L2 of each XCD whose rows are its y-neighbours; by groups, only the 4 halo rows
// of a group are shared with the two neighbouring groups, and the blocks of x-neighbouring planes
// (ng blocks apart) land on the same XCD whenever ng is a multiple of 8.  Same arithmetic as
// g4 (bit-identical results).
// ----------------------------------------------------------------------------------------------
constexpr int kRowsY = 8;

__device__ __forceinline__ double g4v(double m2, double m1, double p1, double p2, double den) {
    double acc = m2;
    acc = acc + (-8.0) * m1;
    acc = acc + 8.0 * p1;
    acc = acc + (-1.0) * p2;
    return acc / den;
}

// the G4 stencil of the LLA kernels: the same sum as g4v, times inv = 1 / (12 h) (a
// multiplication instead of nine divisions per cell)
__device__ __forceinline__ double g4m(double m2, double m1, double p1, double p2, double inv) {
    double acc = m2;
    acc = acc + (-8.0) * m1;
    acc = acc + 8.0 * p1;
    acc = acc + (-1.0) * p2;
    return acc * inv;
}

__device__ __forceinline__ unsigned wrap1(int a, int n) { return (unsigned)(a < 0 ? a + n : (a >= n ? a - n : a)); }

struct RowGroup {
    unsigned x, y0, pl[5], rowy[kRowsY + 4];   // x; first row; planes x-2..x+2; rows y0-2..y0+9 (wrapped)
};

__device__ __forceinline__ RowGroup row_group(Dims d) {
    RowGroup r;
    const unsigned ng = (unsigned)(d.y + kRowsY - 1) / kRowsY;
    r.x = blockIdx.x / ng;
    r.y0 = (blockIdx.x - r.x * ng) * kRowsY;
#pragma unroll
    for (int i = 0; i < 5; ++i) r.pl[i] = wrap1((int)r.x - 2 + i, d.x) * (unsigned)d.y;
#pragma unroll
    for (int i = 0; i < kRowsY + 4; ++i) r.rowy[i] = wrap1((int)r.y0 - 2 + i, d.y);
    return r;
}

__global__ void __launch_bounds__(256) k_grad4_rows(const double* __restrict__ p, Dims d, double h, double scale,
                                                    double* __restrict__ ox, double* __restrict__ oy,
                                                    double* __restrict__ oz) {
    const RowGroup g = row_group(d);
    const double den = 12.0 * h;
    const unsigned nz = (unsigned)d.z;
    for (int z = threadIdx.x; z < d.z; z += blockDim.x) {
        const unsigned zm2 = wrap1(z - 2, d.z), zm1 = wrap1(z - 1, d.z), zp1 = wrap1(z + 1, d.z), zp2 = wrap1(z + 2, d.z);
        double w[kRowsY + 4];
#pragma unroll
        for (int i = 0; i < kRowsY + 4; ++i) w[i] = p[(g.pl[2] + g.rowy[i]) * nz + z];
#pragma unroll
        for (int k = 0; k < kRowsY; ++k) {
            const unsigned y = g.rowy[k + 2];
            const unsigned rc = (g.pl[2] + y) * nz;
            const double gx = g4v(p[(g.pl[0] + y) * nz + z], p[(g.pl[1] + y) * nz + z], p[(g.pl[3] + y) * nz + z],
                                  p[(g.pl[4] + y) * nz + z], den);
            const double gy = g4v(w[k], w[k + 1], w[k + 3], w[k + 4], den);
            const double gz = g4v(p[rc + zm2], p[rc + zm1], p[rc + zp1], p[rc + zp2], den);
            if (g.y0 + k < (unsigned)d.y) {
                ox[rc + z] = scale * gx;
                oy[rc + z] = scale * gy;
                oz[rc + z] = scale * gz;
            }
        }
    }
}

__global__ void __launch_bounds__(256) k_tau_rows(const double* __restrict__ q0, const double* __restrict__ q1,
                                                  const double* __restrict__ q2, Dims d, double h, double post,
                                                  double* __restrict__ tau) {
    const RowGroup g = row_group(d);
    const double den = 12.0 * h;
    const unsigned nz = (unsigned)d.z;
    for (int z = threadIdx.x; z < d.z; z += blockDim.x) {
        const unsigned zm2 = wrap1(z - 2, d.z), zm1 = wrap1(z - 1, d.z), zp1 = wrap1(z + 1, d.z), zp2 = wrap1(z + 2, d.z);
        double w0[kRowsY + 4], w1[kRowsY + 4];
#pragma unroll
        for (int i = 0; i < kRowsY + 4; ++i) {
            w0[i] = q0[(g.pl[2] + g.rowy[i]) * nz + z];
            w1[i] = q1[(g.pl[2] + g.rowy[i]) * nz + z];
        }
#pragma unroll
        for (int k = 0; k < kRowsY; ++k) {
            const unsigned y = g.rowy[k + 2];
            const unsigned rc = (g.pl[2] + y) * nz;
            const double Dxx = g4v(q0[(g.pl[0] + y) * nz + z], q0[(g.pl[1] + y) * nz + z], q0[(g.pl[3] + y) * nz + z],
                                   q0[(g.pl[4] + y) * nz + z], den);
            const double Dyy = g4v(w1[k], w1[k + 1], w1[k + 3], w1[k + 4], den);
            const double Dzz = g4v(q2[rc + zm2], q2[rc + zm1], q2[rc + zp1], q2[rc + zp2], den);
            const double Dyx = g4v(w0[k], w0[k + 1], w0[k + 3], w0[k + 4], den);
            const double Dzx = g4v(q0[rc + zm2], q0[rc + zm1], q0[rc + zp1], q0[rc + zp2], den);
            const double Dzy = g4v(q1[rc + zm2], q1[rc + zm1], q1[rc + zp1], q1[rc + zp2], den);
            double acc = 0.0;
            acc = acc + (Dyy * Dxx - Dyx * Dyx);
            acc = acc + (Dzz * Dxx - Dzx * Dzx);
            acc = acc + (Dzz * Dyy - Dzy * Dzy);
            if (g.y0 + k < (unsigned)d.y) tau[rc + z] = post == 1.0 ? acc : acc * post;
        }
    }
}

// LLA overdensity on a periodic level by groups of rows (the layout of k_grad4_rows): each thread
// takes one z and walks the group's 8 rows; every stencil value is a load at a row base plus z,
// so the per-load index work of the generic kernel (decode, three wraps) is gone.  The same
// operations in the same order as k_lla.
template <bool SUM>
__global__ void __launch_bounds__(256) k_lla_rows(const double* __restrict__ a0, const double* __restrict__ a1,
                                                  const double* __restrict__ a2, const double* __restrict__ b0,
                                                  const double* __restrict__ b1, const double* __restrict__ b2,
                                                  Dims d, double h, double* __restrict__ out) {
    const RowGroup g = row_group(d);
    const double inv = 1.0 / (12.0 * h);
    const unsigned nz = (unsigned)d.z;
    const double* A[3] = {a0, a1, a2};
    const double* Bv[3] = {b0, b1, b2};
    for (int z = threadIdx.x; z < d.z; z += blockDim.x) {
        const unsigned zo[4] = {wrap1(z - 2, d.z), wrap1(z - 1, d.z), wrap1(z + 1, d.z), wrap1(z + 2, d.z)};
        for (int k = 0; k < kRowsY; ++k) {
            if (g.y0 + k >= (unsigned)d.y) break;
            const unsigned y = g.rowy[k + 2];
            const unsigned rc = (g.pl[2] + y) * nz;
            // the four stencil positions along x (planes x-2, x-1, x+1, x+2), y and z
            const unsigned ix[4] = {(g.pl[0] + y) * nz + z, (g.pl[1] + y) * nz + z, (g.pl[3] + y) * nz + z,
                                    (g.pl[4] + y) * nz + z};
            const unsigned iy[4] = {(g.pl[2] + g.rowy[k]) * nz + z, (g.pl[2] + g.rowy[k + 1]) * nz + z,
                                    (g.pl[2] + g.rowy[k + 3]) * nz + z, (g.pl[2] + g.rowy[k + 4]) * nz + z};
            const unsigned iz[4] = {rc + zo[0], rc + zo[1], rc + zo[2], rc + zo[3]};
            double m[3][3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const double* ai = A[i];
                const double* bi = Bv[i];
                auto v = [&](unsigned q) {
                    if constexpr (SUM) return ai[q] + bi[q];
                    else return ai[q];
                };
                m[i][0] = 1.0 * (i == 0) + g4m(v(ix[0]), v(ix[1]), v(ix[2]), v(ix[3]), inv);
                m[i][1] = 1.0 * (i == 1) + g4m(v(iy[0]), v(iy[1]), v(iy[2]), v(iy[3]), inv);
                m[i][2] = 1.0 * (i == 2) + g4m(v(iz[0]), v(iz[1]), v(iz[2]), v(iz[3]), inv);
            }
            const double c0 = m[1][1] * m[2][2] - m[1][2] * m[2][1];
            const double c1 = m[1][0] * m[2][2] - m[1][2] * m[2][0];
            const double c2 = m[1][0] * m[2][1] - m[1][1] * m[2][0];
            const double det = (m[0][0] * c0 - m[0][1] * c1) + m[0][2] * c2;
            out[rc + z] = 1.0 / det - 1.0;
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Large periodic levels by tiles marched along x.  A block owns 16 rows x 64 z of `cx` consecutive
// planes; a thread owns a pair of z-neighbours and keeps their planes x - 2 .. x + 2 of every
// component with an x-stencil in registers.  The y and z stencils of plane x read one slab in LDS:
// every thread writes its own pair of plane x there, and 160 threads a pair of the halo (2 rows and
// 2 cells on each side, without corners), loaded one plane ahead like the own pairs of plane x + 3.
// Two slabs are used in turn, so one barrier per plane orders them.  Per component and cell that is
// 1.125 own loads (cx = 32) and 0.31 halo loads, all of 16 bytes where the arrays allow it.
// Consecutive blocks go to the 8 XCDs in turn, so the tiles are renumbered for each XCD to take a
// contiguous run, whose halos are then its own neighbours' cells (in its L2).  Each kernel has
// the same operations in the same order as its row-group version (bit-identical results).
// Bound: HBM.  Measured at 256^3 (MI355X) against tiles of 4 rows with every slab of the x-window
// in LDS (2.1 loads of 8 bytes per cell): LLA of two sets 328 -> 261 us
// (3.6 TB/s of its compulsory bytes; 154 VGPRs, one block of 8 waves per CU), tau 179 -> 153 us,
// gradient 126 -> 100 us (5.4 TB/s); at 128^3 39 -> 20, 35 -> 20 and 28 -> 15 us.  Tiles of 8 rows (three
// LLA blocks per CU) took 278, 154 and 103 us at 256^3.
// ----------------------------------------------------------------------------------------------
constexpr int kLtY = 16, kLtZ = 64, kLtX = 32, kLtThreads = kLtY * kLtZ / 2;
constexpr int kSZ = kLtZ + 4, kNS = (kLtY + 4) * kSZ;

static bool lpt_tiled(Dims d) {
    return d.x % kLtX == 0 && d.y % kLtY == 0 && d.z % kLtZ == 0 && d.cells() >= ((size_t)1 << 21);
}
// planes per block: two blocks fit a CU, so the march is shortened (at the price of its 4 extra
// planes) until there are 384 blocks or 8 planes are left.  192^3, 432 blocks of 16 planes against 864 of 8:
// gradient 46.6 -> 42.9 us, LLA of one and two sets 88 -> 82 and 109 -> 101 us; 128^3, 128 of 16 against 256
// of 8: gradient 24.6 and 17.9 us
static int tiles_planes(Dims d) {
    const size_t columns = (size_t)(d.y / kLtY) * (size_t)(d.z / kLtZ);
    int cx = kLtX;
    while (cx > 8 && columns * (size_t)(d.x / cx) < 384) cx /= 2;
    return cx;
}
static unsigned tiles_grid(Dims d) {
    return (unsigned)(d.x / tiles_planes(d)) * (unsigned)(d.y / kLtY) * (unsigned)(d.z / kLtZ);
}
static bool pairs_aligned(std::initializer_list<const void*> ps) {
    uintptr_t a = 0;
    for (const void* p : ps) a |= (uintptr_t)p;
    return (a & 15) == 0;
}

template <bool VEC>
__device__ __forceinline__ double2 load_pair(const double* __restrict__ p, unsigned q) {
    if constexpr (VEC) return *(const double2*)(p + q);
    else return make_double2(p[q], p[q + 1]);
}
template <bool VEC>
__device__ __forceinline__ void store_pair(double* __restrict__ p, unsigned q, double2 v) {
    if constexpr (VEC) {
        *(double2*)(p + q) = v;
    } else {
        p[q] = v.x;
        p[q + 1] = v.y;
    }
}

// one component around the thread's pair in the current plane: its slab, the own pair's place in it
// and the own pair's planes x - 2 .. x + 2 (components without an x-stencil: w[2] only)
struct PairView {
    const double* s;
    int me;
    const double2* w;
    __device__ __forceinline__ double2 y(int k) const { return *(const double2*)(s + me + k * kSZ); }
    // the neighbours -2, -1, +1, +2 along z of cell c of the pair
    __device__ __forceinline__ void z(double (*n)[4]) const {
        const double2 l = *(const double2*)(s + me - 2), r = *(const double2*)(s + me + 2), o = w[2];
        n[0][0] = l.x; n[0][1] = l.y; n[0][2] = o.y; n[0][3] = r.x;
        n[1][0] = l.y; n[1][1] = o.x; n[1][2] = r.x; n[1][3] = r.y;
    }
};

// Marches the block's tile: val(c, q) is the pair of component c at linear index q; NW components
// (the first ones) keep an x-window; plane(q, views) computes and stores the pair at q.
template <int NC, int NW, class V, class F>
__device__ __forceinline__ void march_tiles(Dims d, int cx, double (*sl)[NC][kNS], V val, F plane) {
    const unsigned ny = (unsigned)d.y, nz = (unsigned)d.z;
    const unsigned nty = ny / kLtY, ntz = nz / kLtZ;
    unsigned b = blockIdx.x;
    if (gridDim.x % 8 == 0) b = (b % 8) * (gridDim.x / 8) + b / 8;
    const unsigned zt = b % ntz;
    b /= ntz;
    const unsigned yt = b % nty;
    const unsigned x0 = (b / nty) * cx;
    const int tz = (int)(threadIdx.x & 31), ty = (int)(threadIdx.x >> 5);
    const unsigned own = (yt * kLtY + ty) * nz + zt * kLtZ + 2 * tz;
    const int me = (ty + 2) * kSZ + 2 * tz + 2;
    // this thread's pair of the halo: rows -2, -1, 16, 17 (32 pairs each), then the two sides of a row
    const int t = (int)threadIdx.x;
    const bool edge = t < 128 + 2 * kLtY;
    int hy, hz;   // row and cell of the slab
    if (t < 128) {
        hy = (t >> 5) < 2 ? (t >> 5) : (t >> 5) + kLtY;
        hz = 2 * (t & 31) + 2;
    } else {
        hy = ((t - 128) >> 1) + 2;
        hz = t & 1 ? kSZ - 2 : 0;
    }
    if (!edge) hy = hz = 2;   // unused
    const unsigned hoff = wrap1((int)(yt * kLtY) + hy - 2, d.y) * nz + wrap1((int)(zt * kLtZ) + hz - 2, d.z);
    const int hme = hy * kSZ + hz;
    const unsigned np = ny * nz;
    double2 w[NC][5], hv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int k = 0; k < 5; ++k)
            w[c][k] = c < NW || k == 2 ? val(c, wrap1((int)x0 - 2 + k, d.x) * np + own) : make_double2(0.0, 0.0);
        hv[c] = edge ? val(c, x0 * np + hoff) : make_double2(0.0, 0.0);
    }
    for (int i = 0; i < cx; ++i) {
        double (*s)[kNS] = sl[i & 1];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            *(double2*)(s[c] + me) = w[c][2];
            if (edge) *(double2*)(s[c] + hme) = hv[c];
        }
        const bool more = i + 1 < cx;
        double2 nw[NC];
        if (more) {
            const unsigned p1 = wrap1((int)x0 + i + 1, d.x) * np, p3 = wrap1((int)x0 + i + 3, d.x) * np;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                nw[c] = val(c, (c < NW ? p3 : p1) + own);
                if (edge) hv[c] = val(c, p1 + hoff);
            }
        }
        __syncthreads();
        PairView v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = PairView{s[c], me, w[c]};
        plane((x0 + i) * np + own, v);
        if (more)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (c < NW) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) w[c][k] = w[c][k + 1];
                    w[c][4] = nw[c];
                } else {
                    w[c][2] = nw[c];
                }
            }
    }
}

// the block's sum of `acc` to part (or nowhere), waves in order
__device__ __forceinline__ void store_partial(double acc, double* part) {
    __shared__ double s_w[kLtThreads / 64];
    if (!part) return;
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double r = 0.0;
        for (int k = 0; k < kLtThreads / 64; ++k) r += s_w[k];
        part[blockIdx.x] = r;
    }
}

// LLA overdensity (as k_lla_rows); part: the sums of the blocks' results
template <bool SUM, bool VEC>
__global__ void __launch_bounds__(kLtThreads) k_lla_tile(const double* __restrict__ a0, const double* __restrict__ a1,
                                                            const double* __restrict__ a2, const double* __restrict__ b0,
                                                            const double* __restrict__ b1, const double* __restrict__ b2,
                                                            Dims d, int cx, double h, double* __restrict__ out,
                                                            double* __restrict__ part) {
    __shared__ __align__(16) double sl[2][3][kNS];
    const double* A[3] = {a0, a1, a2};
    const double* Bv[3] = {b0, b1, b2};
    const double inv = 1.0 / (12.0 * h);
    auto val = [&](int c, unsigned q) {
        double2 v = load_pair<VEC>(A[c], q);
        if constexpr (SUM) {
            const double2 e = load_pair<VEC>(Bv[c], q);
            v.x = v.x + e.x;
            v.y = v.y + e.y;
        }
        return v;
    };
    double acc = 0.0;
    march_tiles<3, 3>(d, cx, sl, val, [&](unsigned q, const PairView* v) {
        double m[2][3][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double2* w = v[c].w;
            const double2 y0 = v[c].y(-2), y1 = v[c].y(-1), y3 = v[c].y(1), y4 = v[c].y(2);
            double n[2][4];
            v[c].z(n);
            m[0][c][0] = 1.0 * (c == 0) + g4m(w[0].x, w[1].x, w[3].x, w[4].x, inv);
            m[1][c][0] = 1.0 * (c == 0) + g4m(w[0].y, w[1].y, w[3].y, w[4].y, inv);
            m[0][c][1] = 1.0 * (c == 1) + g4m(y0.x, y1.x, y3.x, y4.x, inv);
            m[1][c][1] = 1.0 * (c == 1) + g4m(y0.y, y1.y, y3.y, y4.y, inv);
#pragma unroll
            for (int k = 0; k < 2; ++k) m[k][c][2] = 1.0 * (c == 2) + g4m(n[k][0], n[k][1], n[k][2], n[k][3], inv);
        }
        double o[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const double c0 = m[k][1][1] * m[k][2][2] - m[k][1][2] * m[k][2][1];
            const double c1 = m[k][1][0] * m[k][2][2] - m[k][1][2] * m[k][2][0];
            const double c2 = m[k][1][0] * m[k][2][1] - m[k][1][1] * m[k][2][0];
            const double det = (m[k][0][0] * c0 - m[k][0][1] * c1) + m[k][0][2] * c2;
            o[k] = 1.0 / det - 1.0;
        }
        acc += o[0];
        acc += o[1];
        store_pair<VEC>(out, q, make_double2(o[0], o[1]));
    });
    store_partial(acc, part);
}

// psi_c = scale * G4_c phi (as k_grad4_rows)
template <bool VEC>
__global__ void __launch_bounds__(kLtThreads) k_grad4_tile(const double* __restrict__ p, Dims d, int cx, double h,
                                                           double scale, double* __restrict__ ox,
                                                           double* __restrict__ oy, double* __restrict__ oz) {
    __shared__ __align__(16) double sl[2][1][kNS];
    const double den = 12.0 * h;
    march_tiles<1, 1>(d, cx, sl, [&](int, unsigned q) { return load_pair<VEC>(p, q); },
                      [&](unsigned q, const PairView* v) {
                          const double2* w = v[0].w;
                          const double2 y0 = v[0].y(-2), y1 = v[0].y(-1), y3 = v[0].y(1), y4 = v[0].y(2);
                          double n[2][4];
                          v[0].z(n);
                          store_pair<VEC>(ox, q, make_double2(scale * g4v(w[0].x, w[1].x, w[3].x, w[4].x, den),
                                                              scale * g4v(w[0].y, w[1].y, w[3].y, w[4].y, den)));
                          store_pair<VEC>(oy, q, make_double2(scale * g4v(y0.x, y1.x, y3.x, y4.x, den),
                                                              scale * g4v(y0.y, y1.y, y3.y, y4.y, den)));
                          store_pair<VEC>(oz, q, make_double2(scale * g4v(n[0][0], n[0][1], n[0][2], n[0][3], den),
                                                              scale * g4v(n[1][0], n[1][1], n[1][2], n[1][3], den)));
                      });
}

// tau from the three gradient components (as k_tau_rows); part: the sums of the blocks' results
template <bool VEC>
__global__ void __launch_bounds__(kLtThreads) k_tau_tile(const double* __restrict__ q0, const double* __restrict__ q1,
                                                         const double* __restrict__ q2, Dims d, int cx, double h,
                                                         double post, double* __restrict__ tau,
                                                         double* __restrict__ part) {
    __shared__ __align__(16) double sl[2][3][kNS];
    const double* Q[3] = {q0, q1, q2};
    const double den = 12.0 * h;
    double total = 0.0;
    march_tiles<3, 1>(d, cx, sl, [&](int c, unsigned q) { return load_pair<VEC>(Q[c], q); },
                      [&](unsigned q, const PairView* v) {
                          const double2* w = v[0].w;
                          double2 ya[4], yb[4];
                          double n0[2][4], n1[2][4], n2[2][4], o[2];
#pragma unroll
                          for (int k = 0; k < 4; ++k) {
                              ya[k] = v[0].y(k < 2 ? k - 2 : k - 1);
                              yb[k] = v[1].y(k < 2 ? k - 2 : k - 1);
                          }
                          v[0].z(n0);
                          v[1].z(n1);
                          v[2].z(n2);
#pragma unroll
                          for (int k = 0; k < 2; ++k) {
                              auto at = [&](const double2& e) { return k ? e.y : e.x; };
                              const double Dxx = g4v(at(w[0]), at(w[1]), at(w[3]), at(w[4]), den);
                              const double Dyy = g4v(at(yb[0]), at(yb[1]), at(yb[2]), at(yb[3]), den);
                              const double Dzz = g4v(n2[k][0], n2[k][1], n2[k][2], n2[k][3], den);
                              const double Dyx = g4v(at(ya[0]), at(ya[1]), at(ya[2]), at(ya[3]), den);
                              const double Dzx = g4v(n0[k][0], n0[k][1], n0[k][2], n0[k][3], den);
                              const double Dzy = g4v(n1[k][0], n1[k][1], n1[k][2], n1[k][3], den);
                              double acc = 0.0;
                              acc = acc + (Dyy * Dxx - Dyx * Dyx);
                              acc = acc + (Dzz * Dxx - Dzx * Dzx);
                              acc = acc + (Dzz * Dyy - Dzy * Dzy);
                              o[k] = post == 1.0 ? acc : acc * post;
                              total += o[k];
                          }
                          store_pair<VEC>(tau, q, make_double2(o[0], o[1]));
                      });
    store_partial(total, part);
}

static void run_grad4_tile(const double* p, Dims d, double h, double scale, double* ox, double* oy, double* oz,
                           hipStream_t st) {
    const int cx = tiles_planes(d);
    if (pairs_aligned({p, ox, oy, oz})) k_grad4_tile<true><<<tiles_grid(d), kLtThreads, 0, st>>>(p, d, cx, h, scale, ox, oy, oz);
    else k_grad4_tile<false><<<tiles_grid(d), kLtThreads, 0, st>>>(p, d, cx, h, scale, ox, oy, oz);
}

// the partial sums of a tile kernel's results: wanted, and few enough for the partials buffer
static double* tile_partials(Dims d, double* partials, int* nparts) {
    if (nparts) *nparts = 0;
    if (!partials || tiles_grid(d) > (unsigned)kMaxPartials) return nullptr;
    *nparts = (int)tiles_grid(d);
    return partials;
}

static void run_tau_tile(const double* g0, const double* g1, const double* g2, Dims d, double h, double post,
                         double* tau, double* partials, int* nparts, hipStream_t st) {
    const int cx = tiles_planes(d);
    double* part = tile_partials(d, partials, nparts);
    if (pairs_aligned({g0, g1, g2, tau})) k_tau_tile<true><<<tiles_grid(d), kLtThreads, 0, st>>>(g0, g1, g2, d, cx, h, post, tau, part);
    else k_tau_tile<false><<<tiles_grid(d), kLtThreads, 0, st>>>(g0, g1, g2, d, cx, h, post, tau, part);
}

template <bool SUM>
static void run_lla_tile(const double* const* a, const double* const* b, Dims d, double h, double* out,
                         double* partials, int* nparts, hipStream_t st) {
    const int cx = tiles_planes(d);
    double* part = tile_partials(d, partials, nparts);
    const unsigned g = tiles_grid(d);
    if (pairs_aligned({a[0], a[1], a[2], b[0], b[1], b[2], out}))
        k_lla_tile<SUM, true><<<g, kLtThreads, 0, st>>>(a[0], a[1], a[2], b[0], b[1], b[2], d, cx, h, out, part);
    else
        k_lla_tile<SUM, false><<<g, kLtThreads, 0, st>>>(a[0], a[1], a[2], b[0], b[1], b[2], d, cx, h, out, part);
}

static unsigned rows_grid(Dims d) { return (unsigned)d.x * (unsigned)((d.y + kRowsY - 1) / kRowsY); }
static unsigned rows_block(Dims d) { return d.z >= 256 ? 256u : (unsigned)((d.z + 63) / 64 * 64); }

// padded copy of a patch with width-R tri-quadratic ghosts from its parent
__global__ void k_wide_ghost(const double* __restrict__ pu, const double* __restrict__ u, double* __restrict__ out,
                             Dims d, ParentMap pm, int R, Lay B) {
    const unsigned t = (unsigned)lpt_block() * blockDim.x + threadIdx.x;
    if (t >= (unsigned)B.d.cells()) return;
    int gx, gy, gz;
    decode3(B, t, gx, gy, gz);
    const int i[3] = {gx - R, gy - R, gz - R};
    const int n[3] = {d.x, d.y, d.z};
    if (i[0] >= 0 && i[0] < n[0] && i[1] >= 0 && i[1] < n[1] && i[2] >= 0 && i[2] < n[2]) {
        out[t] = u[((size_t)i[0] * d.y + i[1]) * d.z + i[2]];
        return;
    }
    int P[3];
    double w[3][3];
    for (int a = 0; a < 3; ++a) {
        P[a] = pm.off[a] + (i[a] >> 1);       // floor division, also for negative i
        const double tt = (i[a] & 1) ? 0.25 : -0.25;
        w[a][0] = 0.5 * tt * (tt - 1.0);
        w[a][1] = 1.0 - tt * tt;
        w[a][2] = 0.5 * tt * (tt + 1.0);
    }
    const int pdim[3] = {pm.pl.d.x, pm.pl.d.y, pm.pl.d.z};
    // interpolate along x, then y, then z (tensor product)
    double az = 0.0;
    for (int dz = 0; dz < 3; ++dz) {
        double ay = 0.0;
        for (int dy = 0; dy < 3; ++dy) {
            double ax = 0.0;
            for (int dx = 0; dx < 3; ++dx) {
                int q[3] = {P[0] + dx - 1, P[1] + dy - 1, P[2] + dz - 1};
                if (pm.periodic)
                    for (int k = 0; k < 3; ++k) q[k] = q[k] < 0 ? q[k] + pdim[k] : (q[k] >= pdim[k] ? q[k] - pdim[k] : q[k]);
                ax = ax + w[0][dx] * pu[((size_t)q[0] * pdim[1] + q[1]) * pdim[2] + q[2]];
            }
            ay = ay + w[1][dy] * ax;
        }
        az = az + w[2][dz] * ay;
    }
    out[t] = az;
}

void launch_wide_ghost(const double* pu, const double* u, double* padded, Dims d, ParentMap pm, int R,
                       hipStream_t st) {
    const Lay B(Dims{d.x + 2 * R, d.y + 2 * R, d.z + 2 * R}, 0);
    k_wide_ghost<<<grid_for(B.d.cells()), kBlock, 0, st>>>(pu, u, padded, d, pm, R, B);
}

void launch_grad4(const double* src, int R, Dims d, double h, double scale, double* ox, double* oy, double* oz,
                  hipStream_t st, int order) {
    const Lay B(d, 0);
    if (order == 6) {   // the sixth-order gradient: one thread per cell (periodic, or padded by R >= 3)
        if (R == 0)
            k_grad4<false, 6><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<false>{src, 0, d}, B, h, scale, ox, oy, oz);
        else
            k_grad4<true, 6><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<true>{src, R, d}, B, h, scale, ox, oy, oz);
        return;
    }
    if (R == 0 && lpt_tiled(d))
        run_grad4_tile(src, d, h, scale, ox, oy, oz, st);
    else if (R == 0)
        k_grad4_rows<<<rows_grid(d), rows_block(d), 0, st>>>(src, d, h, scale, ox, oy, oz);
    else
        k_grad4<true><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<true>{src, R, d}, B, h, scale, ox, oy, oz);
}

void launch_tau(const double* src, int R, Dims d, double h, double* tau, double* psi, hipStream_t st, int order,
                double* partials, int* nparts) {
    if (nparts) *nparts = 0;
    const int rg = order / 2;   // the gradient's radius
    const int e = R >= rg ? R - rg : 0;
    const Lay E(Dims{d.x + 2 * e, d.y + 2 * e, d.z + 2 * e}, 0);
    const Lay B(d, 0);
    double* p0 = psi;
    double* p1 = psi + E.d.cells();
    double* p2 = psi + 2 * E.d.cells();
    if (order == 6) {   // the sixth-order gradient twice: one thread per cell
        if (R == 0) {
            k_psi<false, 6><<<grid_for(E.d.cells()), kBlock, 0, st>>>(Src<false>{src, 0, d}, E, 0, h, p0, p1, p2);
            k_tau_psi<false, 6><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<false>{p0, 0, d}, Src<false>{p1, 0, d},
                                                                        Src<false>{p2, 0, d}, B, h, 1.0, tau);
        } else {
            k_psi<true, 6><<<grid_for(E.d.cells()), kBlock, 0, st>>>(Src<true>{src, R, d}, E, e, h, p0, p1, p2);
            k_tau_psi<true, 6><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<true>{p0, e, d}, Src<true>{p1, e, d},
                                                                       Src<true>{p2, e, d}, B, h, 1.0, tau);
        }
        return;
    }
    if (R == 0) {
        k_psi<false><<<grid_for(E.d.cells()), kBlock, 0, st>>>(Src<false>{src, 0, d}, E, 0, h, p0, p1, p2);
        if (lpt_tiled(d)) run_tau_tile(p0, p1, p2, d, h, 1.0, tau, partials, nparts, st);
        else k_tau_rows<<<rows_grid(d), rows_block(d), 0, st>>>(p0, p1, p2, d, h, 1.0, tau);
    } else {
        k_psi<true><<<grid_for(E.d.cells()), kBlock, 0, st>>>(Src<true>{src, R, d}, E, e, h, p0, p1, p2);
        k_tau_psi<true><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<true>{p0, e, d}, Src<true>{p1, e, d},
                                                                Src<true>{p2, e, d}, B, h, 1.0, tau);
    }
}

void launch_tau_from_grad(const double* g0, const double* g1, const double* g2, Dims d, double h, double post,
                         double* tau, hipStream_t st, int order, double* partials, int* nparts) {
    if (nparts) *nparts = 0;
    if (order == 6) {
        k_tau_psi<false, 6><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<false>{g0, 0, d}, Src<false>{g1, 0, d},
                                                                    Src<false>{g2, 0, d}, Lay(d, 0), h, post, tau);
        return;
    }
    if (lpt_tiled(d)) run_tau_tile(g0, g1, g2, d, h, post, tau, partials, nparts, st);
    else k_tau_rows<<<rows_grid(d), rows_block(d), 0, st>>>(g0, g1, g2, d, h, post, tau);
}


void launch_lla(const double* const* a, const double* const* b, int R, Dims d, double h, double* out, hipStream_t st,
                double* partials, int* nparts) {
    if (nparts) *nparts = 0;
    const Lay B(d, 0);
    const int sum = b != nullptr;
    const double* const* bb = sum ? b : a;
    // periodic levels (every base here has at least 2 cells per axis, so a single wrap of an
    // offset of 2 holds) by x-marched tiles where they divide the level, else by groups of rows;
    // padded patches by the per-cell kernel
    if (R == 0 && lpt_tiled(d)) {
        if (sum) run_lla_tile<true>(a, bb, d, h, out, partials, nparts, st);
        else run_lla_tile<false>(a, bb, d, h, out, partials, nparts, st);
    } else if (R == 0 && sum)
        k_lla_rows<true><<<rows_grid(d), rows_block(d), 0, st>>>(a[0], a[1], a[2], bb[0], bb[1], bb[2], d, h, out);
    else if (R == 0)
        k_lla_rows<false><<<rows_grid(d), rows_block(d), 0, st>>>(a[0], a[1], a[2], bb[0], bb[1], bb[2], d, h, out);
    else
        k_lla<true><<<grid_for(d.cells()), kBlock, 0, st>>>(Src<true>{a[0], R, d}, Src<true>{a[1], R, d},
                                                           Src<true>{a[2], R, d}, Src<true>{bb[0], R, d},
                                                           Src<true>{bb[1], R, d}, Src<true>{bb[2], R, d}, sum, B, h,
                                                           out);
}

void launch_add2(const double* a, const double* b, double* dst, size_t n, hipStream_t st) {
    k_add2<<<grid_for(n), kBlock, 0, st>>>(a, b, dst, n);
}

}  // namespace mgic
