// Two red-black sweeps of the smoother (Section 3.2, steps 2 and 9) in one launch, for periodic
// colour-split power-of-two levels of at least 64^3 cells.
//
// As four launches the sweeps move 6 words per cell (every half-sweep reads the other colour, f and
// writes its own).  One pass needs 2.5: the black half of u (the first red half-sweep reads nothing
// else), f, and both colours written.  A block owns kRows rows x 64 z of `cx` consecutive planes and
// a halo of four cells, and marches along x with the four half-sweeps staggered by a plane:
//   plane p: red from the old black;      plane p - 1: black from that red;
//   plane p - 2: red from that black;     plane p - 3: black from that red.
// A thread owns a run of W = 16 / sizeof(T) cells of each colour in one row of the tile (halo
// included) and keeps the planes that its own updates need in registers: the x-neighbours are its own
// values of the plane before and after, the cell's z-neighbours lie in the other colour's run.  The y
// rows beside it and the one z-neighbour outside the run come from LDS, where every thread leaves what
// it has just formed for the next step (two buffers, one barrier per step).  Values in the outer layers of
// the tile are wrong after the half-sweeps that reach beyond it, one layer each, and are never stored.
// Halo cells are recomputed by the neighbouring tiles, and the result goes to a second array, so no block
// reads what another writes.  Every value is formed by the operations of the one-step kernels in their
// order: the bits are the same.
//
// Mode kSweepPlain: u as it is.  kSweepCorr: the coarse-grid correction (step 8) is added to the black
// values as they are read (nothing else reads it).  kSweepRed: the first red half-sweep is already done
// (by the fused outer step); the red values are read instead of the black ones.
//
// Bound: HBM at 512^3, the Infinity Cache and FP64/FP32 arithmetic (recomputed halos) below.  Measured
// (MI355X) against four half-sweep launches, plain / with the correction (there prolongation and first
// half-sweep were one pass in FP32, two in FP64 from 256^3): 512^3 FP64 1528 -> 586 / 1783 -> 708 us (4.6
// TB/s of the compulsory bytes; a plain 1 GiB copy reaches 5.0), FP32 600 -> 363 / 695 -> 479 us; 256^3 FP64
// 134 -> 82 / 163 -> 103 us, FP32 66 -> 38 / 74 -> 48 us; 128^3 FP64 22 -> 19 / 23 -> 23 us, FP32 20 -> 14
// / 20 -> 17 us.  A 64^3 level has only 16 such blocks and stays with half-sweeps.

#include <hip/hip_ext.h>

#include <type_traits>

#include "mg_internal.h"
#include "p2_bodies.h"

namespace mgic {

namespace {

constexpr int kRows = 32;                 // rows of a tile
constexpr int kZ = 64;                    // z cells of a tile
constexpr int kHalo = 4;                  // rows on each side: one per half-sweep

template <class T>
struct SweepTile {
    static constexpr int W = Vec16<T>::W;
    static constexpr int kRuns = kZ / (2 * W) + 2;   // runs of a row, one of halo on each side (at least 4 cells)
    static constexpr int kNy = kRows + 2 * kHalo;
    static constexpr int kCells = kNy * kRuns;       // threads with a run
    static constexpr int kThreads = (kCells + 63) / 64 * 64;
};

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

template <class T, int MODE>
__global__ void __launch_bounds__(SweepTile<T>::kThreads)
k_two_sweeps(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ out, int lg, int cx, T h2,
             const T* __restrict__ pu, const T* __restrict__ uold) {
    using TL = SweepTile<T>;
    using V = V16<T>;
    constexpr int W = TL::W, NR = TL::kRuns;
    __shared__ V lds[2][4][TL::kCells];   // [buffer][half-sweep whose input it is][row * NR + run]
    const unsigned n = 1u << lg, m = n - 1, nzh = n >> 1;
    // tiles by planes, rows, z; each XCD takes a contiguous run of them, so that the halos of a chunk of
    // planes are in its own L2
    unsigned b = blockIdx.x;
    if (gridDim.x % 8 == 0) b = (b % 8) * (gridDim.x / 8) + b / 8;
    const unsigned ntz = n / kZ, nty = n / kRows;
    const unsigned zt = b % ntz;
    b /= ntz;
    const unsigned y0 = (b % nty) * kRows;
    const int x0 = (int)(b / nty) * cx;
    // idle threads of the last wave shadow the last run (they store nothing)
    const int t = min((int)threadIdx.x, TL::kCells - 1);
    const int r = t / NR, k = t - r * NR;
    const bool mine = (int)threadIdx.x < TL::kCells && r >= kHalo && r < kHalo + kRows && k >= 1 && k < NR - 1;
    const bool live = (int)threadIdx.x < TL::kCells;
    const unsigned y = (y0 + (unsigned)(r - kHalo)) & m;
    const unsigned j0 = (zt * (kZ / 2) + (unsigned)((k - 1) * W)) & (nzh - 1);
    const unsigned at = (y << lg) + j0;              // the red run of plane 0; the black one nzh further
    const int up = (r > 0 ? -NR : 0), dn = (r < TL::kNy - 1 ? NR : 0);
    const int lf = (k > 0 ? -1 : 0), rt = (k < NR - 1 ? 1 : 0);
    auto plane = [&](int x) { return ((unsigned)x & m) << (2 * lg); };
    auto load_start = [&](int x) -> V {              // the half-sweeps' start: the black run (MODE red: the red run)
        const unsigned p = plane(x) + at;
        if constexpr (MODE == kSweepRed) return *(const V*)(u + p);
        V v = *(const V*)(u + p + nzh);
        if constexpr (MODE == kSweepCorr) {
            T d[W], o[W];
            corr_delta<T>(pu, uold, lg - 1, ((unsigned)x & m) >> 1, y >> 1, j0, d);
#pragma unroll
            for (int i = 0; i < W; ++i) o[i] = lane<T>(v, i) + d[i];
            v = pack<T>(o);
        }
        return v;
    };
    auto load_f = [&](int x, unsigned half) { return *(const V*)(f + plane(x) + at + half); };
    // rings of four planes, plane x in slot (x - x0 + 8) & 3 (a constant in the unrolled steps)
    V s0[4], r1[4], b1[4], r2[4], fr[4], fb[4];
    const int first = x0 - 3;                        // plane of the first half-sweep in step 0
    // step s works on p = first + s; slot of plane first + s + d: (s + d) & 3
#pragma unroll
    for (int i = 0; i < 4; ++i) s0[i] = r1[i] = b1[i] = r2[i] = fr[i] = fb[i] = V{};
    s0[3] = load_start(first - 1);
    s0[0] = load_start(first);
    s0[1] = load_start(first + 1);
    fr[0] = load_f(first, 0);
    fb[3] = load_f(first - 1, nzh);
    lds[0][0][t] = MODE == kSweepRed ? V{} : s0[0];
    lds[0][1][t] = lds[0][2][t] = lds[0][3][t] = V{};
    if constexpr (MODE == kSweepRed) {
        r1[3] = s0[3];
        lds[0][1][t] = r1[3];
    }
    __syncthreads();
    const int steps = cx + 6;
    const unsigned par = (unsigned)(first + 8) + y;   // parity of red cells in plane p: (par + s) & 1
    auto half = [&](int buf, int st, const V& xm, const V& xp, const V& c, const V& fv, bool q) -> V {
        const V* L = lds[buf][st];
        const V ym = L[t + up], yp = L[t + dn];
        const T* e = (const T*)(L + (q ? t + rt : t + lf));
        const T edge = q ? e[0] : e[W - 1];
        return update_run<T>(xm, xp, ym, yp, c, edge, fv, q, h2);
    };
    auto step = [&](int s, auto phase) {
        constexpr int P = decltype(phase)::value;     // s & 3
        constexpr int a0 = P & 3, am1 = (P + 3) & 3, am2 = (P + 2) & 3, am3 = (P + 1) & 3, ap1 = (P + 1) & 3,
                      ap2 = (P + 2) & 3;
        constexpr int rd = P & 1, wr = rd ^ 1;
        const int p = first + s;
        const bool odd = (par + (unsigned)s) & 1u;    // z parity of the red cells of plane p
        const bool more = s + 1 < steps;
        // slots that this step fills early hold planes that it still reads: load into locals
        V ns, nfr, nfb;
        if (more) {
            ns = load_start(p + 2);
            nfr = load_f(p + 1, 0);
            nfb = load_f(p, nzh);
        }
        // red of plane p, black of p - 1, red of p - 2, black of p - 3
        if constexpr (MODE == kSweepRed) r1[a0] = s0[a0];
        else r1[a0] = half(rd, 0, s0[am1], s0[ap1], s0[a0], fr[a0], odd);
        b1[am1] = half(rd, 1, r1[am2], r1[a0], r1[am1], fb[am1], odd);        // black of p - 1: parity as red of p
        const V rn = half(rd, 2, b1[am3], b1[am1], b1[am2], fr[am2], odd);
        const V bn = half(rd, 3, r2[P & 3], rn, r2[am3], fb[am3], odd);       // slot P holds red of p - 4
        r2[am2] = rn;
        if (mine) {
            const int xr = p - 2, xb = p - 3;
            if (xr >= x0 && xr < x0 + cx) *(V*)(out + plane(xr) + at) = rn;
            if (xb >= x0) *(V*)(out + plane(xb) + at + nzh) = bn;
        }
        if (live) {
            if constexpr (MODE != kSweepRed) lds[wr][0][t] = s0[ap1];
            lds[wr][1][t] = r1[a0];
            lds[wr][2][t] = b1[am1];
            lds[wr][3][t] = rn;
        }
        if (more) {
            s0[ap2] = ns;
            fr[ap1] = nfr;
            fb[a0] = nfb;
        }
        __syncthreads();
    };
    int s = 0;
    for (; s + 4 <= steps; s += 4) {
        step(s, std::integral_constant<int, 0>{});
        step(s + 1, std::integral_constant<int, 1>{});
        step(s + 2, std::integral_constant<int, 2>{});
        step(s + 3, std::integral_constant<int, 3>{});
    }
    if (s < steps) step(s, std::integral_constant<int, 0>{});
    if (s + 1 < steps) step(s + 1, std::integral_constant<int, 1>{});
    if (s + 2 < steps) step(s + 2, std::integral_constant<int, 2>{});
}

// planes per block: about one block per CU, at least 8 planes (the march has 6 more)
int sweep_planes(int n) {
    const int columns = (n / kRows) * (n / kZ);
    int cx = n;
    while (cx > 8 && columns * (n / cx) < 256) cx /= 2;
    return cx;
}

}  // namespace

bool two_sweeps_ok(const Lay& L) {
    return L.pow2 && L.split && L.lgx == L.lgy && L.lgy == L.lgz && L.lgz >= 7 && L.lgz <= 10;
}

template <class T>
void launch_two_sweeps(const T* u, const T* f, T* out, const Lay& L, double h, int mode, const T* pu, const T* uold,
                       hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const int n = L.d.x, cx = sweep_planes(n);
    const dim3 grid((unsigned)((n / kRows) * (n / kZ) * (n / cx))), block(SweepTile<T>::kThreads);
    const T h2 = (T)(h * h);
    auto run = [&](auto kernel) {
        if (ev0) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev0, ev1, 0, u, f, out, L.lgx, cx, h2, pu, uold);
        else kernel<<<grid, block, 0, st>>>(u, f, out, L.lgx, cx, h2, pu, uold);
    };
    if (mode == kSweepPlain) run(k_two_sweeps<T, kSweepPlain>);
    else if (mode == kSweepCorr) run(k_two_sweeps<T, kSweepCorr>);
    else run(k_two_sweeps<T, kSweepRed>);
}

template void launch_two_sweeps<float>(const float*, const float*, float*, const Lay&, double, int, const float*,
                                       const float*, hipStream_t, hipEvent_t, hipEvent_t);
template void launch_two_sweeps<double>(const double*, const double*, double*, const Lay&, double, int,
                                        const double*, const double*, hipStream_t, hipEvent_t, hipEvent_t);

}  // namespace mgic
