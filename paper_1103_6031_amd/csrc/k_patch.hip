// Two red-black sweeps of a refinement patch in one launch, its ghost zones formed on the chip.
//
// One half-sweep of a patch needs the ghosts of its colour's face cells, and these the patch's two layers
// along the face as they then are, so two sweeps took four ghost fills and four half-sweeps: at 128^3 eight
// launches of 4 - 6 us for 25 MB each, bound by launches and their drain.  Here a block takes a tile of
// 16 x 16 rows and 2 kOwn runs with its halo - four rows, one 16-byte run - into LDS, both colours, and does
// all four half-sweeps there, its halo shrinking by a row each (the next tile recomputes those values).  A
// ghost lies in the LDS cell just outside the patch, where the half-sweep looks for it; before each half-sweep
// every 2 x 2 group of face cells in the tile forms its four ghosts from the tile's own cells and the parent's
// part, which its thread has formed once and keeps in registers (tile origins and halos are even, so no group
// is cut).  The result goes to a second array.  Every value is formed by the operations of the one-step
// kernels in their order: the bits are the same.
//
// CORR: the coarse-grid correction (step 8) is added as the patch is read.  Otherwise (before the coarse-grid
// visit) the ghosts of the result are written too: the residual reads them.
//
// Bound: latency of the phases (load, ten barriers, store) up to one tile per CU, LDS traffic of the recomputed
// halo above.  Measured (MI355X) per V-cycle, both passes, against 8 half-sweeps, 9 ghost fills and the
// prolongation: FP32 64^3 60 -> 33 us, 96^3 80 -> 35, 128^3 95 -> 36, 160^3 130 -> 69, 240^3 283 -> 226;
// FP64 64^3 60 -> 30 us, 96^3 99 -> 31, 128^3 110 -> 60, 160^3 165 -> 111, 240^3 389 -> 435.

#include <hip/hip_ext.h>

#include "ghost_bodies.h"
#include "mg_internal.h"
#include "p2_bodies.h"
#include "sweep_bodies.h"

namespace mgic {

namespace {

constexpr int kTile = 16;                   // own rows in x and in y
constexpr int kOwn = 4;                     // own runs of each colour per row
constexpr int kEdge = kTile + 8;            // rows with the halo
constexpr int kRuns = kOwn + 2;             // runs with the halo
constexpr int kCells = kEdge * kEdge * kRuns;
constexpr int kThreads = 1024;
constexpr int kLoad = (kCells + kThreads - 1) / kThreads;
constexpr int kInner = kEdge - 2;           // rows that are updated at all
constexpr int kUpd = (kInner * kInner * kRuns + kThreads - 1) / kThreads;
static_assert(kTile * kTile * kOwn == kThreads, "one own run of each colour per thread");

template <class T, bool CORR>
__global__ void __launch_bounds__(kThreads)
k_patch_sweeps(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ out, T* __restrict__ g, Lay L, T h2,
               const T* __restrict__ pu, const T* __restrict__ uold, ParentMap pm) {
    using V = V16<T>;
    constexpr int W = Vec16<T>::W;
    constexpr int RZ = 2 * W * kRuns;       // z extent with the halo
    __shared__ V lds[2 * kCells];
    const Dims d = L.d;
    const int n[3] = {d.x, d.y, d.z};
    const unsigned nzh = (unsigned)d.z >> 1;
    // each XCD takes a contiguous run of tiles, so that the halos of neighbours are in its own L2
    unsigned b = blockIdx.x;
    b = (b % 8) * (gridDim.x / 8) + min(b % 8, gridDim.x % 8) + b / 8;
    const int tz = (d.z + 2 * W * kOwn - 1) / (2 * W * kOwn), ty = (d.y + kTile - 1) / kTile;
    const int o[3] = {(int)(b / (unsigned)(ty * tz)) * kTile, (int)(b / (unsigned)tz % (unsigned)ty) * kTile,
                      (int)(b % (unsigned)tz) * 2 * W * kOwn};           // first own cell
    const int r0[3] = {o[0] - 4, o[1] - 4, o[2] - 2 * W};               // first cell with the halo
    const int t = (int)threadIdx.x;

    // the tile's both colours; f of the runs that this thread updates.  (Runs outside the patch read its first
    // one: no branch, so that all loads are in flight together.)
    V vr[kLoad], vb[kLoad];
    [[maybe_unused]] V co[kLoad];
    [[maybe_unused]] T cp[kLoad][W];
#pragma unroll
    for (int i = 0; i < kLoad; ++i) {
        const int c = t + i * kThreads, row = c / kRuns, k = c - row * kRuns;
        int x = r0[0] + row / kEdge, y = r0[1] + row % kEdge, z = r0[2] + 2 * W * k;
        if (x < 0 || x >= d.x || y < 0 || y >= d.y || z < 0 || z >= d.z) x = y = z = 0;
        const size_t p = ((size_t)x * d.y + y) * d.z + (z >> 1);
        vr[i] = *(const V*)(u + p);
        vb[i] = *(const V*)(u + p + nzh);
        if constexpr (CORR) {   // cell z = 2 j + q of either colour lies in coarse cell j
            co[i] = *(const V*)(uold + ((size_t)(x >> 1) * (d.y >> 1) + (y >> 1)) * nzh + (z >> 1));
#pragma unroll
            for (int m = 0; m < W; ++m) cp[i][m] = pu[pidx(pm, x >> 1, y >> 1, (z >> 1) + m)];
        }
    }
    V fr[kUpd], fb[kUpd];
    int at[kUpd], depth[kUpd];              // LDS run, and the number of half-sweeps that update it
    bool odd[kUpd];                         // the red cells of the row have odd z
#pragma unroll
    for (int i = 0; i < kUpd; ++i) {
        const int c = t + i * kThreads, row = c / kRuns, k = c - row * kRuns;
        const int lx = 1 + row / kInner, ly = 1 + row % kInner;
        int x = r0[0] + lx, y = r0[1] + ly, z = r0[2] + 2 * W * k;
        const bool in = c < kInner * kInner * kRuns && x >= 0 && x < d.x && y >= 0 && y < d.y && z >= 0 && z < d.z;
        at[i] = (lx * kEdge + ly) * kRuns + k;
        depth[i] = in ? min(min(lx, kEdge - 1 - lx), min(ly, kEdge - 1 - ly)) : 0;
        odd[i] = (x + y) & 1;
        if (!in) x = y = z = 0;
        const size_t p = ((size_t)x * d.y + y) * d.z + (z >> 1);
        fr[i] = *(const V*)(f + p);
        fb[i] = *(const V*)(f + p + nzh);
    }
#pragma unroll
    for (int i = 0; i < kLoad; ++i) {
        const int c = t + i * kThreads;
        if constexpr (CORR) {
            T a[W], e[W];
#pragma unroll
            for (int m = 0; m < W; ++m) {
                const T dl = cp[i][m] - lane<T>(co[i], m);
                a[m] = lane<T>(vr[i], m) + dl;
                e[m] = lane<T>(vb[i], m) + dl;
            }
            vr[i] = pack<T>(a);
            vb[i] = pack<T>(e);
        }
        if (c < kCells) {
            lds[c] = vr[i];
            lds[kCells + c] = vb[i];
        }
    }
    // the groups of face cells with the halo: at most two per thread
    int lo[3], m[3];
    constexpr int R[3] = {kEdge, kEdge, RZ};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = max(r0[a], 0) >> 1;
        m[a] = (min(r0[a] + R[a], n[a]) >> 1) - lo[a];
    }
    constexpr int G = 2;
    static_assert(4 * (kEdge / 2) * (RZ / 2) + 2 * (kEdge / 2) * (kEdge / 2) <= G * kThreads, "groups of a tile");
    double aq[G][4], O[G];
    int face[G], gJ[G], gK[G];
    int groups = 0;
#pragma unroll
    for (int i = 0; i < G; ++i) face[i] = -1;
#pragma unroll
    for (int fc = 0; fc < 6; ++fc) {
        const int a = fc >> 1, bb = a == 0 ? 1 : 0, cc = a == 2 ? 1 : 2;
        if (fc & 1 ? n[a] >= r0[a] + R[a] : r0[a] >= 0) continue;   // no updated cell of the tile is at this face
        const int cnt = m[bb] * m[cc];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int k = t + i * kThreads - groups;
            if (k >= 0 && k < cnt) {
                face[i] = fc;
                gJ[i] = lo[bb] + k / m[cc];
                gK[i] = lo[cc] + k % m[cc];
            }
        }
        groups += cnt;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (face[i] < 0) continue;
        double P[3][3];
        ghost_parent(pu, pm, d, face[i], gJ[i], gK[i], P);
#pragma unroll
        for (int q = 0; q < 4; ++q) aq[i][q] = ghost_interp(P, q >> 1, q & 1);
        O[i] = P[1][1];
    }
    __syncthreads();

    // entry of cell (x, y, z), or of the ghost there
    T* cell = (T*)lds;
    auto entry = [&](int x, int y, int z) -> T& {
        const int row = (x - r0[0]) * kEdge + (y - r0[1]);
        return cell[(((x + y + z) & 1) * kCells + row * kRuns) * W + ((z - r0[2]) >> 1)];
    };
    // ghost of face cell (x, y, z)
    auto ghost_at = [&](int fc, int x, int y, int z) -> T& {
        const int a = fc >> 1, s = fc & 1 ? 1 : -1;
        return entry(x + (a == 0 ? s : 0), y + (a == 1 ? s : 0), z + (a == 2 ? s : 0));
    };
    auto ghosts = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (face[i] < 0) continue;
            const int a = face[i] >> 1, side = face[i] & 1;
            const int na = pick(a, d.x, d.y, d.z), i0 = side ? na - 1 : 0, i1 = side ? na - 2 : 1;
            double u0[4], u1[4], g0[4];
            int px[4], py[4], pz[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int J = 2 * gJ[i] + (q >> 1), K = 2 * gK[i] + (q & 1);
                px[q] = a == 0 ? i0 : J;
                py[q] = a == 1 ? i0 : (a == 0 ? J : K);
                pz[q] = a == 2 ? i0 : K;
                u0[q] = (double)entry(px[q], py[q], pz[q]);
                u1[q] = (double)entry(a == 0 ? i1 : px[q], a == 1 ? i1 : py[q], a == 2 ? i1 : pz[q]);
                g0[q] = ghost_g0(aq[i][q], u0[q], u1[q]);
            }
            auto mean4 = [](const double* v) { return ((v[0] + v[1]) + (v[2] + v[3])) * 0.25; };
            const double shift = ghost_shift(mean4(u0), mean4(u1), mean4(g0), O[i]);
#pragma unroll
            for (int q = 0; q < 4; ++q) ghost_at(face[i], px[q], py[q], pz[q]) = (T)(g0[q] + shift);
        }
    };
    auto half = [&](int s) __attribute__((always_inline)) {               // half-sweep s of the four: red, black, red, black
        if (groups) {
            ghosts();
            __syncthreads();
        }
        V* own = lds + (s & 1) * kCells;
        const V* oth = lds + ((s & 1) ^ 1) * kCells;
#pragma unroll
        for (int i = 0; i < kUpd; ++i) {
            if (depth[i] <= s) continue;
            const int c = at[i];
            const bool q = odd[i] != (bool)(s & 1);
            const T edge = *((const T*)(oth + c) + (q ? W : -1));
            own[c] = update_run<T>(oth[c - kEdge * kRuns], oth[c + kEdge * kRuns], oth[c - kRuns], oth[c + kRuns],
                                   oth[c], edge, s & 1 ? fb[i] : fr[i], q, h2);
        }
        __syncthreads();
    };
    half(0);
    half(1);
    half(2);
    half(3);
    {
        const int row = t / kOwn, k = t - row * kOwn;
        const int lx = row / kTile, ly = row % kTile;
        const int x = o[0] + lx, y = o[1] + ly, z = o[2] + 2 * W * k;
        if (x < d.x && y < d.y && z < d.z) {
            const int c = ((lx + 4) * kEdge + ly + 4) * kRuns + k + 1;
            const size_t p = ((size_t)x * d.y + y) * d.z + (z >> 1);
            *(V*)(out + p) = lds[c];
            *(V*)(out + p + nzh) = lds[kCells + c];
        }
    }
    if constexpr (!CORR) {
        ghosts();
        // (each thread reads back what it has written: the groups of this tile's own cells)
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (face[i] < 0) continue;
            const int fc = face[i], a = fc >> 1, i0 = fc & 1 ? pick(a, d.x, d.y, d.z) - 1 : 0;
            const size_t fx = (size_t)d.y * d.z, fy = (size_t)d.x * d.z, fz = (size_t)d.x * d.y;
            T* p = g + (fc < 2 ? fc * fx : (fc < 4 ? 2 * fx + (fc - 2) * fy : 2 * (fx + fy) + (fc - 4) * fz));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int J = 2 * gJ[i] + (q >> 1), K = 2 * gK[i] + (q & 1);
                const int x = a == 0 ? i0 : J, y = a == 1 ? i0 : (a == 0 ? J : K), z = a == 2 ? i0 : K;
                if (x >= o[0] && x < o[0] + kTile && y >= o[1] && y < o[1] + kTile && z >= o[2] &&
                    z < o[2] + 2 * W * kOwn)
                    p[(size_t)J * (a == 2 ? d.y : d.z) + K] = ghost_at(fc, x, y, z);
            }
        }
    }
}

}  // namespace

// FP64 tiles own half the cells in z (the halo is 3.4 times the tile's work): not above 2^23 cells, where the
// one-step launches are bound by memory and cost less (figures above)
bool patch_sweeps_ok(const Lay& L, size_t elem) {
    const int W = (int)(16 / elem);
    return (elem == 4 || L.d.cells() <= (size_t)1 << 23) && L.split && L.d.x % 2 == 0 && L.d.y % 2 == 0 && L.d.z % (2 * W) == 0;
}

template <class T>
void launch_patch_sweeps(const T* u, const T* f, T* out, T* ghosts, const Lay& L, double h, bool corr, const T* pu,
                         const T* uold, const ParentMap& pm, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    auto tiles = [](int n, int t) { return (unsigned)((n + t - 1) / t); };
    const dim3 grid(tiles(L.d.x, kTile) * tiles(L.d.y, kTile) * tiles(L.d.z, 2 * Vec16<T>::W * kOwn)), block(kThreads);
    const T h2 = (T)(h * h);
    auto run = [&](auto kernel) {
        if (ev0) hipExtLaunchKernelGGL(kernel, grid, block, 0, st, ev0, ev1, 0, u, f, out, ghosts, L, h2, pu, uold, pm);
        else kernel<<<grid, block, 0, st>>>(u, f, out, ghosts, L, h2, pu, uold, pm);
    };
    if (corr) run(k_patch_sweeps<T, true>);
    else run(k_patch_sweeps<T, false>);
}

template void launch_patch_sweeps<float>(const float*, const float*, float*, float*, const Lay&, double, bool,
                                         const float*, const float*, const ParentMap&, hipStream_t, hipEvent_t,
                                         hipEvent_t);
template void launch_patch_sweeps<double>(const double*, const double*, double*, double*, const Lay&, double, bool,
                                          const double*, const double*, const ParentMap&, hipStream_t, hipEvent_t,
                                          hipEvent_t);

}  // namespace mgic
