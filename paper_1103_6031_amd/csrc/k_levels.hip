// Fused small-level kernels of the FAS V-cycle (Section 3.2) for the periodic coarsenings of 16^3
// to 64^3 cells.
//
// As one-step kernels each such level costs eleven launches per cycle (FAS right-hand side,
// 2 nu1 half-sweeps, residual + restriction, prolongation, 2 nu2 half-sweeps), and at these sizes
// every launch costs about its dispatch latency.  Here one workgroup per 8^3 tile holds the tile
// and a halo in LDS and runs a whole leg of the cycle there:
//   pre:  FAS right-hand side (step 6 of the parent), nu1 red-black sweeps (step 2), residual and
//         restriction (steps 3-5) of the tile;
//   post: coarse-grid correction (step 8), nu2 red-black sweeps (step 9) of the tile.
// A half-sweep of a cell needs its neighbours' previous values, so after each half-sweep the
// region that is still exact shrinks by one cell; the halo is as deep as the number of
// half-sweeps (plus one for the residual stencil), and the halo cells are computed redundantly
// by the neighbouring tiles.  Every value is formed by the same operations in the same order as
// in the one-step kernels, so the results are bit-identical to them.  Workgroups read the level's
// arrays and write a second copy (no workgroup reads what another writes).
//
// Edges that are no power of two (20, 24, 28, 40, 48, 56: bases of 3, 5 or 7 times one) take the
// same kernels with multiplications and one conditional wrap in place of shifts and masks; where 8
// does not divide the edge, the last tile of a row ends inside the level.  Measured for a 96^3 base, nu (1, 2),
// whose 48^3 and 24^3 levels the legs run, per V-cycle of the solve: mixed 112 -> 88 us, FP64 124 -> 102 us (MI355X).

#include <hip/hip_ext.h>

#include <type_traits>

#include "mg_internal.h"
#include "p2_bodies.h"

namespace mgic {

constexpr int kTile = 8;            // tile edge (cells)
constexpr int kFusedThreads = 512;  // one thread per tile cell

// LDS cells of the legs' u regions (f = 0) and f regions (f = 1)
constexpr int cube(int s) { return s * s * s; }
constexpr int pre_cells(int nu, int f) { return cube(kTile + 2 * (2 * nu + 1) - 2 * f); }
constexpr int post_cells(int nu, int f) { return cube(kTile + 2 * (2 * nu) - 2 * f); }

// Loops over the cells of a region: each thread takes the cells t = threadIdx.x + r * 512; every
// pass first forms all its values (an index past the end is clamped to the last cell, so every
// load stays inside the arrays) and only then stores them, so that the loads of all passes are in
// flight together.
template <int N>
struct Passes {
    static constexpr int n = (N + kFusedThreads - 1) / kFusedThreads;
    __device__ static int cell(int r) {
        const int t = (int)threadIdx.x + r * kFusedThreads;
        return t < N ? t : N - 1;
    }
    __device__ static bool live(int r) { return N % kFusedThreads == 0 || (int)threadIdx.x + r * kFusedThreads < N; }
};

// one red-black half-sweep of `colour` over the cells of [k, S - k)^3 of an S^3 LDS region of u
// (origin parity p0: the cell (i, j, m) has colour (i + j + m + p0) & 1); f is the (S - 2)^3
// region one cell inside it.  The cells of one colour read only the other colour, so all new
// values are formed before any is stored.
template <class T, int S, int k>
__device__ __forceinline__ void lds_half_sweep(T* su, const T* sf, T h2, int colour, int p0) {
    constexpr int W = S - 2 * k, Wh = W / 2, SF = S - 2;
    using Pp = Passes<W * W * Wh>;
    T v[Pp::n];
    int at[Pp::n];
#pragma unroll
    for (int r = 0; r < Pp::n; ++r) {
        const int t = Pp::cell(r);
        const int row = t / Wh, m = t - row * Wh;
        const int i = k + row / W, j = k + row % W;
        const int q = (i + j + k + p0 + colour) & 1;
        const int z = k + 2 * m + q;
        const int c = (i * S + j) * S + z;
        const T s = ((su[c - S * S] + su[c + S * S]) + (su[c - S] + su[c + S])) + (su[c - 1] + su[c + 1]);
        v[r] = div6(s - h2 * sf[((i - 1) * SF + (j - 1)) * SF + (z - 1)]);
        at[r] = c;
    }
#pragma unroll
    for (int r = 0; r < Pp::n; ++r)
        if (Pp::live(r)) su[at[r]] = v[r];
}

template <class T, int S, int k, int kend>
__device__ __forceinline__ void lds_sweeps(T* su, const T* sf, T h2, int p0) {
    if constexpr (k <= kend) {
        lds_half_sweep<T, S, k>(su, sf, h2, (k - 1) & 1, p0);   // red (0) first
        __syncthreads();
        lds_sweeps<T, S, k + 1, kend>(su, sf, h2, p0);
    }
}

// Index arithmetic of a level of edge n (even) and its tiles: P2 for n = 2^lg.
template <bool P2>
struct LevelIdx {
    int n, lg;
    // origin of tile b
    __device__ __forceinline__ void origin(unsigned b, int& ox, int& oy, int& oz) const {
        if constexpr (P2) {
            const int lt = lg - 3;
            ox = (int)(b >> (2 * lt)) * kTile;
            oy = (int)((b >> lt) & ((1u << lt) - 1)) * kTile;
            oz = (int)(b & ((1u << lt) - 1)) * kTile;
        } else {
            const unsigned nt = (unsigned)(n + kTile - 1) / kTile, r = b / nt, q = r / nt;
            ox = (int)q * kTile;
            oy = (int)(r - q * nt) * kTile;
            oz = (int)(b - r * nt) * kTile;
        }
    }
    // periodic wrap of a coordinate in -n .. 2 n - 1
    __device__ __forceinline__ unsigned wrap(int a) const {
        if constexpr (P2) return (unsigned)a & ((1u << lg) - 1);
        else return (unsigned)(a < 0 ? a + n : (a >= n ? a - n : a));
    }
    __device__ __forceinline__ bool inside(int x, int y, int z) const { return P2 || (x < n && y < n && z < n); }
    // position in the colour-split level, in the colour-split coarse level, and in the coarse level's
    // natural order
    __device__ __forceinline__ unsigned at(unsigned x, unsigned y, unsigned z) const {
        if constexpr (P2) return sidx(lg, x, y, z);
        else return (x * n + y) * n + (((x + y + z) & 1u) ? (unsigned)n >> 1 : 0u) + (z >> 1);
    }
    __device__ __forceinline__ unsigned coarse(unsigned X, unsigned Y, unsigned Z) const {
        if constexpr (P2) return sidx(lg - 1, X, Y, Z);
        const unsigned c = (unsigned)n >> 1;
        return (X * c + Y) * c + (((X + Y + Z) & 1u) ? c >> 1 : 0u) + (Z >> 1);
    }
    __device__ __forceinline__ unsigned natural(unsigned X, unsigned Y, unsigned Z) const {
        if constexpr (P2) return (((X << (lg - 1)) | Y) << (lg - 1)) | Z;
        const unsigned c = (unsigned)n >> 1;
        return (X * c + Y) * c + Z;
    }
};

// v[S^3 region with origin o - R] = a[cell] (periodic wrap), into LDS
template <class T, int S, bool P2>
__device__ __forceinline__ void load_region(T* dst, const T* __restrict__ a, LevelIdx<P2> ix, int ox, int oy, int oz,
                                            int R) {
    using Pp = Passes<S * S * S>;
    T v[Pp::n];
#pragma unroll
    for (int r = 0; r < Pp::n; ++r) {
        const int t = Pp::cell(r);
        const int i = t / (S * S), j = (t / S) % S, m = t % S;
        v[r] = a[ix.at(ix.wrap(ox - R + i), ix.wrap(oy - R + j), ix.wrap(oz - R + m))];
    }
#pragma unroll
    for (int r = 0; r < Pp::n; ++r)
        if (Pp::live(r)) dst[(int)threadIdx.x + r * kFusedThreads] = v[r];
}

// pre leg on a level of edge ix.n: u, f are the level's arrays as the parent's restriction left
// them; uo, fo receive the smoothed u and the FAS right-hand side of this tile; pu, pf, uold the
// restricted u, the restricted residual and its copy for the coarse level
template <class T, int NU, bool P2>
__device__ __forceinline__ void body_level_pre(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ uo,
                                               T* __restrict__ fo, T* __restrict__ pu, T* __restrict__ pf,
                                               T* __restrict__ uold, LevelIdx<P2> ix, T h2, unsigned b, T* su,
                                               T* sf) {
    constexpr int R = 2 * NU + 1;      // u halo: 2 nu1 half-sweeps + the residual stencil
    constexpr int S = kTile + 2 * R, SF = S - 2;
    int ox, oy, oz;
    ix.origin(b, ox, oy, oz);
    load_region<T, S, P2>(su, u, ix, ox, oy, oz, R);
    load_region<T, SF, P2>(sf, f, ix, ox, oy, oz, R - 1);
    __syncthreads();
    // FAS right-hand side on the f region: f += L u (u here is the restricted fine u)
    {
        using Pp = Passes<SF * SF * SF>;
        T v[Pp::n];
#pragma unroll
        for (int r = 0; r < Pp::n; ++r) {
            const int t = Pp::cell(r);
            const int i = t / (SF * SF), j = (t / SF) % SF, m = t % SF;
            const int c = ((i + 1) * S + (j + 1)) * S + (m + 1);
            const T s = ((su[c - S * S] + su[c + S * S]) + (su[c - S] + su[c + S])) + (su[c - 1] + su[c + 1]);
            v[r] = sf[t] + (s - T(6) * su[c]) / h2;
        }
#pragma unroll
        for (int r = 0; r < Pp::n; ++r)
            if (Pp::live(r)) sf[(int)threadIdx.x + r * kFusedThreads] = v[r];
    }
    __syncthreads();
    lds_sweeps<T, S, 1, 2 * NU>(su, sf, h2, R & 1);
    // residual and restriction of the tile's 4^3 coarse cells: each thread one child, the 8
    // children of a coarse cell in 8 neighbouring lanes, summed in the order (a, b, e)
    {
        const int t = threadIdx.x, ch = t & 7, cc = t >> 3;
        const int X = cc >> 4, Y = (cc >> 2) & 3, Z = cc & 3;
        const int x = 2 * X + (ch >> 2), y = 2 * Y + ((ch >> 1) & 1), z = 2 * Z + (ch & 1);
        const int c = ((x + R) * S + (y + R)) * S + (z + R);
        const T ui = su[c];
        const T fi = sf[((x + R - 1) * SF + (y + R - 1)) * SF + (z + R - 1)];
        const T s = ((su[c - S * S] + su[c + S * S]) + (su[c - S] + su[c + S])) + (su[c - 1] + su[c + 1]);
        const T lap = (s - T(6) * ui) / h2;
        const T r = fi - lap;
        const int lane0 = (int)(threadIdx.x & 63) & ~7;
        T sr = T(0), sum_u = T(0);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            sr = sr + __shfl(r, lane0 + q, 64);
            sum_u = sum_u + __shfl(ui, lane0 + q, 64);
        }
        if (!ix.inside(ox + x, oy + y, oz + z)) return;   // all 8 children or none: the edge is even
        if (ch == 0) {
            const unsigned Xg = (unsigned)(ox / 2 + X), Yg = (unsigned)(oy / 2 + Y), Zg = (unsigned)(oz / 2 + Z);
            const T uc = sum_u * T(0.125);
            const unsigned P = ix.coarse(Xg, Yg, Zg);
            pu[P] = uc;
            pf[P] = sr * T(0.125);
            uold[ix.natural(Xg, Yg, Zg)] = uc;
        }
        // the tile itself: smoothed u and the FAS right-hand side
        const unsigned g = ix.at((unsigned)(ox + x), (unsigned)(oy + y), (unsigned)(oz + z));
        uo[g] = ui;
        fo[g] = fi;
    }
}

template <class T, int NU, bool P2>
__global__ void __launch_bounds__(kFusedThreads)
k_level_pre(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ uo, T* __restrict__ fo,
            T* __restrict__ pu, T* __restrict__ pf, T* __restrict__ uold, LevelIdx<P2> ix, T h2) {
    __shared__ T su[pre_cells(NU, 0)], sf[pre_cells(NU, 1)];
    body_level_pre<T, NU, P2>(u, f, uo, fo, pu, pf, uold, ix, h2, blockIdx.x, su, sf);
}

// post leg: u = ui + (uc[parent] - uold[parent]) over the tile and a halo of 2 nu2 cells, then
// nu2 red-black sweeps; the tile is written to uout.  fi is the FAS right-hand side of the level.
template <class T, int NU, bool P2>
__device__ __forceinline__ void body_level_post(const T* __restrict__ ui, const T* __restrict__ fi,
                                                const T* __restrict__ uc, const T* __restrict__ uold,
                                                T* __restrict__ uout, LevelIdx<P2> ix, T h2, unsigned b, T* su,
                                                T* sf) {
    constexpr int R = 2 * NU;
    constexpr int S = kTile + 2 * R, SF = S - 2;
    int ox, oy, oz;
    ix.origin(b, ox, oy, oz);
    {
        using Pp = Passes<S * S * S>;
        T v[Pp::n];
#pragma unroll
        for (int r = 0; r < Pp::n; ++r) {
            const int t = Pp::cell(r);
            const int i = t / (S * S), j = (t / S) % S, m = t % S;
            const unsigned x = ix.wrap(ox - R + i), y = ix.wrap(oy - R + j), z = ix.wrap(oz - R + m);
            const unsigned X = x >> 1, Y = y >> 1, Z = z >> 1;
            v[r] = ui[ix.at(x, y, z)] + (uc[ix.coarse(X, Y, Z)] - uold[ix.natural(X, Y, Z)]);
        }
#pragma unroll
        for (int r = 0; r < Pp::n; ++r)
            if (Pp::live(r)) su[(int)threadIdx.x + r * kFusedThreads] = v[r];
    }
    load_region<T, SF, P2>(sf, fi, ix, ox, oy, oz, R - 1);
    __syncthreads();
    lds_sweeps<T, S, 1, 2 * NU>(su, sf, h2, R & 1);
    {
        const int t = threadIdx.x;
        const int x = t >> 6, y = (t >> 3) & 7, z = t & 7;
        if (ix.inside(ox + x, oy + y, oz + z))
            uout[ix.at((unsigned)(ox + x), (unsigned)(oy + y), (unsigned)(oz + z))] =
                su[((x + R) * S + (y + R)) * S + (z + R)];
    }
}

template <class T, int NU, bool P2>
__global__ void __launch_bounds__(kFusedThreads)
k_level_post(const T* __restrict__ ui, const T* __restrict__ fi, const T* __restrict__ uc,
             const T* __restrict__ uold, T* __restrict__ uout, LevelIdx<P2> ix, T h2) {
    __shared__ T su[post_cells(NU, 0)], sf[post_cells(NU, 1)];
    body_level_post<T, NU, P2>(ui, fi, uc, uold, uout, ix, h2, blockIdx.x, su, sf);
}

// The same legs of the levels of many batched instances: a block finds its instance's level and
// tile.  pre: a = {u, f, uo, pu, pf, uold}, part = fo; post: a = {ui, fi, uc, uold, uout}.
template <class T, int NU>
__global__ void __launch_bounds__(kFusedThreads) kb_level_pre(const BSeg* __restrict__ segs, int nseg,
                                                              const int* __restrict__ active) {
    __shared__ T su[pre_cells(NU, 0)], sf[pre_cells(NU, 1)];
    unsigned lb;
    const BSeg& s = seg_of(segs, nseg, lb);
    if (!active[s.inst]) return;
    const int n = s.L.d.x, lg = s.L.lgx;
    const T h2 = (T)(s.h * s.h);
    const T *u = (const T*)s.a[0], *f = (const T*)s.a[1];
    T *uo = (T*)s.a[2], *pu = (T*)s.a[3], *pf = (T*)s.a[4], *uold = (T*)s.a[5], *fo = (T*)s.part;
    if (lg >= 0) body_level_pre<T, NU, true>(u, f, uo, fo, pu, pf, uold, LevelIdx<true>{n, lg}, h2, lb, su, sf);
    else body_level_pre<T, NU, false>(u, f, uo, fo, pu, pf, uold, LevelIdx<false>{n, lg}, h2, lb, su, sf);
}

template <class T, int NU>
__global__ void __launch_bounds__(kFusedThreads) kb_level_post(const BSeg* __restrict__ segs, int nseg,
                                                               const int* __restrict__ active) {
    __shared__ T su[post_cells(NU, 0)], sf[post_cells(NU, 1)];
    unsigned lb;
    const BSeg& s = seg_of(segs, nseg, lb);
    if (!active[s.inst]) return;
    const int n = s.L.d.x, lg = s.L.lgx;
    const T h2 = (T)(s.h * s.h);
    const T *ui = (const T*)s.a[0], *fi = (const T*)s.a[1], *uc = (const T*)s.a[2], *uold = (const T*)s.a[3];
    T* uout = (T*)s.a[4];
    if (lg >= 0) body_level_post<T, NU, true>(ui, fi, uc, uold, uout, LevelIdx<true>{n, lg}, h2, lb, su, sf);
    else body_level_post<T, NU, false>(ui, fi, uc, uold, uout, LevelIdx<false>{n, lg}, h2, lb, su, sf);
}

// ----------------------------------------------------------------------------------------------
// One-step transfer kernels for periodic colour-split power-of-two cubes (the larger levels of a
// power-of-two base), with the same arithmetic as the generic ones and coalesced accesses: the
// lanes of a wave take consecutive coarse cells Z of a row, whose fine cells sit at consecutive
// positions of the fine half-rows.
// ----------------------------------------------------------------------------------------------

// Block order of the power-of-two kernels on large levels (the 16-byte half-sweeps and the
// residual-restriction).  Consecutive blocks go to the 8 XCDs in turn, so the rows at the edges
// of a block's run were fetched again into another XCD's L2 by the neighbouring blocks (counters
// at 256^3: 1.09x the compulsory bytes for the half-sweep, 1.22x for the residual-restriction).
// Within each group of 32 blocks the order is permuted so that 4 consecutive runs share an XCD
// (hardware block b takes run 4 (b mod 8) + (b div 8) mod 4); the interleave across XCDs stays
// fine-grained.  Applied only where an x plane spans a multiple of 32 blocks, so that
// x-neighbouring planes keep sharing an XCD (at 128^3 a half-sweep plane is 8 blocks, and the
// permutation measured slower there).  Measured at 256^3: half-sweep counters 1.02x, FP32
// 16.7 -> 16.4 us; residual-restriction fetch -15%, FP32 26.0 -> 24.8 us.
__device__ __forceinline__ unsigned xcd_quads(unsigned b, unsigned grid, unsigned blocks_per_plane) {
    if (grid % 32 != 0 || blocks_per_plane % 32 != 0) return b;
    return (b & ~31u) | (((b & 7u) << 2) | ((b >> 3) & 3u));
}

// steps 3-5, one thread per coarse cell (cell_resid_restrict_p2)
template <class T>
__global__ void __launch_bounds__(256)
k_resid_restrict_p2(const T* __restrict__ u, const T* __restrict__ f, int lg, T h2, T* __restrict__ pu,
                    T* __restrict__ pf, T* __restrict__ uold) {
    const int lc = lg - 1;
    const unsigned t = xcd_quads(blockIdx.x, gridDim.x, (1u << (2 * lc)) / blockDim.x) * blockDim.x + threadIdx.x;
    if (t >= 1u << (3 * lc)) return;
    cell_resid_restrict_p2<T>(u, f, lg, h2, pu, pf, uold, t);
}

// step 8 on the black cells: the black cell (row, j) of a fine row lies in the parent (X, Y, j)
template <class T>
__global__ void __launch_bounds__(256)
k_prolong_black_p2(T* __restrict__ u, int lg, const T* __restrict__ pu, const T* __restrict__ uold) {
    const int lc = lg - 1;
    const unsigned nzh = 1u << lc, m = (1u << lg) - 1;
    const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 1u << (3 * lg - 1)) return;
    const unsigned row = t >> lc, j = t & (nzh - 1);
    const unsigned x = row >> lg, y = row & m;
    const unsigned X = x >> 1, Y = y >> 1;
    const unsigned i = (row << lg) + nzh + j;
    u[i] = u[i] + (pu[sidx(lc, X, Y, j)] - uold[(((X << lc) | Y) << lc) | j]);
}

// step 6 on a whole periodic coarse level (edge 2^lg): f += L u for the cell t (natural order)
template <class T>
__global__ void __launch_bounds__(256)
k_fas_rhs_p2(const T* __restrict__ pu, T* __restrict__ pf, int lg, T H2) {
    const unsigned m = (1u << lg) - 1;
    const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= 1u << (3 * lg)) return;
    const unsigned x = t >> (2 * lg), y = (t >> lg) & m, z = t & m;
    const unsigned i = sidx(lg, x, y, z);
    const T s = ((pu[sidx(lg, (x - 1) & m, y, z)] + pu[sidx(lg, (x + 1) & m, y, z)]) +
                 (pu[sidx(lg, x, (y - 1) & m, z)] + pu[sidx(lg, x, (y + 1) & m, z)])) +
                (pu[sidx(lg, x, y, (z - 1) & m)] + pu[sidx(lg, x, y, (z + 1) & m)]);
    pf[i] = pf[i] + (s - T(6) * pu[i]) / H2;
}

template <class T>
void launch_resid_restrict_p2(const T* u, const T* f, int n, double h, T* pu, T* pf, T* uold, hipStream_t st) {
    const int lg = __builtin_ctz((unsigned)n);
    const unsigned cells = 1u << (3 * (lg - 1));
    k_resid_restrict_p2<T><<<(cells + 255) / 256, 256, 0, st>>>(u, f, lg, (T)(h * h), pu, pf, uold);
}

// step 8 on the black cells, W at a time with 16-byte accesses (run_prolong_black_vec)
template <class T>
__global__ void __launch_bounds__(256)
k_prolong_black_vec(T* __restrict__ u, int lg, const T* __restrict__ pu, const T* __restrict__ uold) {
    constexpr int W = Vec16<T>::W;
    const unsigned ch = blockIdx.x * blockDim.x + threadIdx.x;
    if (ch < (1u << (3 * lg - 1 - __builtin_ctz(W)))) run_prolong_black_vec<T>(u, lg, pu, uold, ch);
}

template <class T>
void launch_prolong_black_p2(T* u, int n, const T* pu, const T* uold, hipStream_t st) {
    constexpr int W = Vec16<T>::W;
    const int lg = __builtin_ctz((unsigned)n);
    const unsigned cells = 1u << (3 * lg - 1);
    if ((1u << (lg - 1)) % W == 0) {   // half-rows hold whole runs
        const unsigned runs = cells / W;
        k_prolong_black_vec<T><<<(runs + 255) / 256, 256, 0, st>>>(u, lg, pu, uold);
    } else {
        k_prolong_black_p2<T><<<(cells + 255) / 256, 256, 0, st>>>(u, lg, pu, uold);
    }
}

template <class T>
void launch_fas_rhs_p2(const T* pu, T* pf, int n, double H, hipStream_t st) {
    const int lg = __builtin_ctz((unsigned)n);
    const unsigned cells = 1u << (3 * lg);
    k_fas_rhs_p2<T><<<(cells + 255) / 256, 256, 0, st>>>(pu, pf, lg, (T)(H * H));
}

// ----------------------------------------------------------------------------------------------
// Red-black half-sweep on a periodic colour-split power-of-two level with 16-byte accesses: a
// thread takes W = 16 / sizeof(T) consecutive cells j0 .. j0 + W - 1 of its colour in one
// half-row (4 FP32 or 2 FP64 cells) and reads each neighbour run, f and the other colour's entries
// of its own row as one vector; the one z-neighbour outside that run (entry j0 - 1 or j0 + W of
// the other half, by the row's parity) is a scalar load.  Each cell is updated with the
// expression of cell_rbgs_split, so the bits are the same.
// ----------------------------------------------------------------------------------------------
template <class T, int CH>
__global__ void __launch_bounds__(256)
k_rbgs_vec(T* __restrict__ u, const T* __restrict__ f, int lgx, int lgy, int lgz, T h2, int colour) {
    constexpr int W = Vec16<T>::W;
    const unsigned lzh = (unsigned)lgz - 1;
    const unsigned chunks = 1u << (lgx + lgy + lzh - __builtin_ctz(W));   // W-cell runs of one colour
    const unsigned bl = xcd_quads(blockIdx.x, gridDim.x, (1u << (lgy + lzh - __builtin_ctz(W))) / (CH * blockDim.x));
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const unsigned ch = (bl * CH + c) * blockDim.x + threadIdx.x;
        if (ch >= chunks) break;
        run_rbgs_vec<T>(u, f, lgx, lgy, lgz, h2, colour, ch);
    }
}

// The first red half-sweep after the coarse-grid correction (step 8 then step 9), in one pass:
// the correction u += pu[parent] - uold[parent] of the black cells is only ever read by this
// half-sweep (the black half-sweep after it rewrites every black cell without reading it), so it
// is applied here to each black value as it is read, and never stored.  A black cell (row, j) of
// the fine level lies in the parent (x >> 1, y >> 1, j); the parents of a run of W black cells are
// W consecutive Z of one coarse row: a vector of uold (natural order) and two half-vectors of pu
// (colour-split order, even and odd Z in the two halves).  Same arithmetic as k_prolong_black_p2
// followed by k_rbgs_vec, so the same bits.
template <class T>
__global__ void __launch_bounds__(256)
k_rbgs_vec_corr(T* __restrict__ u, const T* __restrict__ f, int lgx, int lgy, int lgz, T h2,
                const T* __restrict__ pu, const T* __restrict__ uold) {
    using V = typename Vec16<T>::type;
    constexpr int W = Vec16<T>::W;
    const unsigned lzh = (unsigned)lgz - 1, nzh = 1u << lzh, mx = (1u << lgx) - 1, my = (1u << lgy) - 1;
    const int lc = lgz - 1;                        // the coarse level is a cube of edge 2^(lgz - 1)
    const unsigned chunks = 1u << (lgx + lgy + lzh - __builtin_ctz(W));
    const unsigned bl = xcd_quads(blockIdx.x, gridDim.x, (1u << (lgy + lzh - __builtin_ctz(W))) / blockDim.x);
    const unsigned ch = bl * blockDim.x + threadIdx.x;
    if (ch >= chunks) return;
    const unsigned t = ch * W, row = t >> lzh, j0 = t & (nzh - 1);
    const unsigned x = row >> lgy, y = row & my;
    const unsigned q = (x + y) & 1u;              // z parity of red cells in the row
    const unsigned r0 = row << lgz;
    const unsigned xm = (x - 1) & mx, xp = (x + 1) & mx, ym = (y - 1) & my, yp = (y + 1) & my;
    // the black runs read are those of rows x-1, x+1, y-1, y+1 and the own row; their parents lie in
    // the own parent row (X, Y) and in one more row along x (for x-1 if x is even, else x+1) and
    // one along y, so three correction runs cover all five
    const unsigned X = x >> 1, Y = y >> 1;
    T dO[W], dX[W], dY[W];
    corr_delta<T>(pu, uold, 1 << lc, X, Y, j0, dO);
    corr_delta<T>(pu, uold, 1 << lc, ((x & 1u) ? xp : xm) >> 1, Y, j0, dX);
    corr_delta<T>(pu, uold, 1 << lc, X, ((y & 1u) ? yp : ym) >> 1, j0, dY);
    auto run = [&](unsigned xr, unsigned yr, const T* d, T* c) {
        const V v = *(const V*)(u + (((xr << lgy) | yr) << lgz) + nzh + j0);
#pragma unroll
        for (int k = 0; k < W; ++k) c[k] = lane<T>(v, k) + d[k];
    };
    T XM[W], XP[W], YM[W], YP[W], C[W];
    run(xm, y, (x & 1u) ? dO : dX, XM);
    run(xp, y, (x & 1u) ? dX : dO, XP);
    run(x, ym, (y & 1u) ? dO : dY, YM);
    run(x, yp, (y & 1u) ? dY : dO, YP);
    run(x, y, dO, C);
    // the one black entry of the own row outside the run (j0 - 1 or j0 + W, by parity), corrected
    const unsigned je = q ? ((j0 + W) & (nzh - 1)) : ((j0 - 1) & (nzh - 1));
    T edge;
    {
        const unsigned ncz = 1u << lc, rb = ((X << lc) | Y) << lc;
        edge = u[r0 + nzh + je] + (pu[rb + ((X + Y + je) & 1u) * (ncz >> 1) + (je >> 1)] - uold[rb + je]);
    }
    const V F = *(const V*)(f + r0 + j0);
    T out[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
        const T zm = q ? C[k] : (k == 0 ? edge : C[k - 1]);
        const T zp = q ? (k == W - 1 ? edge : C[k + 1]) : C[k];
        const T s = ((XM[k] + XP[k]) + (YM[k] + YP[k])) + (zm + zp);
        out[k] = div6(s - h2 * lane<T>(F, k));
    }
    V o;
    if constexpr (W == 4) o = V{out[0], out[1], out[2], out[3]};
    else o = V{out[0], out[1]};
    *(V*)(u + r0 + j0) = o;
}

template <class T>
void launch_rbgs_vec_corr(T* u, const T* f, const Lay& L, double h, const T* pu, const T* uold, hipStream_t st) {
    constexpr int W = Vec16<T>::W;
    const unsigned chunks = (unsigned)(L.d.cells() / 2 / W);
    k_rbgs_vec_corr<T><<<(chunks + 255) / 256, 256, 0, st>>>(u, f, L.lgx, L.lgy, L.lgz, (T)(h * h), pu, uold);
}

// Step 6 on a whole periodic colour-split power-of-two level with 16-byte accesses (run_fas_vec:
// a thread takes the runs j0 .. j0 + W - 1 of both colours of one row).
template <class T>
__global__ void __launch_bounds__(256)
k_fas_vec(const T* __restrict__ pu, T* __restrict__ pf, int lg, T H2) {
    constexpr int W = Vec16<T>::W;
    const unsigned chunks = 1u << (3 * lg - 1 - __builtin_ctz(W));   // runs per colour
    const unsigned ch = blockIdx.x * blockDim.x + threadIdx.x;
    if (ch < chunks) run_fas_vec<T>(pu, pf, lg, H2, ch);
}

template <class T>
void launch_fas_vec(const T* pu, T* pf, int n, double H, hipStream_t st) {
    constexpr int W = Vec16<T>::W;
    const int lg = __builtin_ctz((unsigned)n);
    const unsigned chunks = (unsigned)((size_t)n * n * n / 2 / W);
    k_fas_vec<T><<<(chunks + 255) / 256, 256, 0, st>>>(pu, pf, lg, (T)(H * H));
}

bool rbgs_vec_ok(const Lay& L, size_t elem) {
    const unsigned W = 16u / (unsigned)elem;
    return L.pow2 && L.split && L.lgz >= 1 && ((1u << (L.lgz - 1)) % W) == 0;
}

template <class T>
void launch_rbgs_vec(T* u, const T* f, const Lay& L, double h, int colour, hipStream_t st, hipEvent_t ev0,
                     hipEvent_t ev1) {
    constexpr int W = Vec16<T>::W;
    const unsigned chunks = (unsigned)(L.d.cells() / 2 / W);
    const T h2 = (T)(h * h);
    // measured: 1 run per thread is best for FP32 at 128^3 and 256^3 and for FP64 at 128^3; FP64
    // at 256^3 and above is 5% faster with 2
    // stamped by the events when they are given (kernel timing), else a plain launch (the form
    // captured into graphs)
    if (sizeof(T) == 8 && chunks >= (1u << 22)) {
        if (ev0)
            hipExtLaunchKernelGGL(k_rbgs_vec<T, 2>, dim3((chunks + 511) / 512), dim3(256), 0, st, ev0, ev1, 0, u, f,
                                  L.lgx, L.lgy, L.lgz, h2, colour);
        else
            k_rbgs_vec<T, 2><<<(chunks + 511) / 512, 256, 0, st>>>(u, f, L.lgx, L.lgy, L.lgz, h2, colour);
    } else {
        if (ev0)
            hipExtLaunchKernelGGL(k_rbgs_vec<T, 1>, dim3((chunks + 255) / 256), dim3(256), 0, st, ev0, ev1, 0, u, f,
                                  L.lgx, L.lgy, L.lgz, h2, colour);
        else
            k_rbgs_vec<T, 1><<<(chunks + 255) / 256, 256, 0, st>>>(u, f, L.lgx, L.lgy, L.lgz, h2, colour);
    }
}

bool level_fusable(int n, int nu1, int nu2) {
    // colour-split with a colour-split coarse level; the wrap of LevelIdx needs n > kTile + 5
    return n >= 16 && n <= 64 && n % 4 == 0 && nu1 >= 1 && nu1 <= 2 && nu2 >= 1 && nu2 <= 2;
}

unsigned level_tiles(int n) {
    const unsigned t = (unsigned)(n + kTile - 1) / kTile;
    return t * t * t;
}

template <class T>
void launch_level_pre(const T* u, const T* f, T* uo, T* fo, T* pu, T* pf, T* uold, int n, double h, int nu1,
                      hipStream_t st) {
    const int lg = log2_exact(n);
    const unsigned tiles = level_tiles(n);
    const T h2 = (T)(h * h);
    auto run = [&](auto ix) {
        constexpr bool P2 = std::is_same_v<decltype(ix), LevelIdx<true>>;
        if (nu1 == 1) k_level_pre<T, 1, P2><<<tiles, kFusedThreads, 0, st>>>(u, f, uo, fo, pu, pf, uold, ix, h2);
        else k_level_pre<T, 2, P2><<<tiles, kFusedThreads, 0, st>>>(u, f, uo, fo, pu, pf, uold, ix, h2);
    };
    if (lg >= 0) run(LevelIdx<true>{n, lg});
    else run(LevelIdx<false>{n, lg});
}

template <class T>
void launch_level_post(const T* ui, const T* fi, const T* uc, const T* uold, T* uout, int n, double h, int nu2,
                       hipStream_t st) {
    const int lg = log2_exact(n);
    const unsigned tiles = level_tiles(n);
    const T h2 = (T)(h * h);
    auto run = [&](auto ix) {
        constexpr bool P2 = std::is_same_v<decltype(ix), LevelIdx<true>>;
        if (nu2 == 1) k_level_post<T, 1, P2><<<tiles, kFusedThreads, 0, st>>>(ui, fi, uc, uold, uout, ix, h2);
        else k_level_post<T, 2, P2><<<tiles, kFusedThreads, 0, st>>>(ui, fi, uc, uold, uout, ix, h2);
    };
    if (lg >= 0) run(LevelIdx<true>{n, lg});
    else run(LevelIdx<false>{n, lg});
}

template <class T>
void launch_b_level_pre(const BSeg* segs, int nseg, unsigned grid, const int* active, int nu1, hipStream_t st) {
    if (nu1 == 1) kb_level_pre<T, 1><<<grid, kFusedThreads, 0, st>>>(segs, nseg, active);
    else kb_level_pre<T, 2><<<grid, kFusedThreads, 0, st>>>(segs, nseg, active);
}

template <class T>
void launch_b_level_post(const BSeg* segs, int nseg, unsigned grid, const int* active, int nu2, hipStream_t st) {
    if (nu2 == 1) kb_level_post<T, 1><<<grid, kFusedThreads, 0, st>>>(segs, nseg, active);
    else kb_level_post<T, 2><<<grid, kFusedThreads, 0, st>>>(segs, nseg, active);
}

#define MG_INST(T)                                                                                      \
    template void launch_resid_restrict_p2<T>(const T*, const T*, int, double, T*, T*, T*, hipStream_t);      \
    template void launch_prolong_black_p2<T>(T*, int, const T*, const T*, hipStream_t);                       \
    template void launch_fas_rhs_p2<T>(const T*, T*, int, double, hipStream_t);                               \
    template void launch_rbgs_vec<T>(T*, const T*, const Lay&, double, int, hipStream_t, hipEvent_t, hipEvent_t); \
    template void launch_rbgs_vec_corr<T>(T*, const T*, const Lay&, double, const T*, const T*, hipStream_t);     \
    template void launch_fas_vec<T>(const T*, T*, int, double, hipStream_t);                                  \
    template void launch_level_pre<T>(const T*, const T*, T*, T*, T*, T*, T*, int, double, int, hipStream_t); \
    template void launch_level_post<T>(const T*, const T*, const T*, const T*, T*, int, double, int, hipStream_t); \
    template void launch_b_level_pre<T>(const BSeg*, int, unsigned, const int*, int, hipStream_t);            \
    template void launch_b_level_post<T>(const BSeg*, int, unsigned, const int*, int, hipStream_t);
MG_INST(float)
MG_INST(double)
#undef MG_INST

}  // namespace mgic
