// Two red-black sweeps of the smoother (Section 3.2, steps 2 and 9) in one launch, for periodic
// colour-split levels of 16^3 to 1024^3 cells (two_sweeps_ok; below 17^3 the single-workgroup tail takes them).
//
// As four launches the sweeps move 6 words per cell (every half-sweep reads the other colour, f and
// writes its own).  One pass needs 2.5: the black half of u (the first red half-sweep reads nothing
// else), f, and both colours written.  A block owns a tile of rows and z of `cx` consecutive planes and
// a halo of four cells (one run in z), and marches along x with the four half-sweeps staggered by a plane:
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
// Bound: HBM at 512^3, the Infinity Cache and FP64/FP32 arithmetic (recomputed halos) below, the latency of
// a step (0.6 - 0.8 us) on levels of few tiles.  Measured (MI355X) against four half-sweep launches, plain /
// with the correction (there prolongation and first half-sweep were one pass in FP32, two in FP64 from 256^3):
// 512^3 FP64 1528 -> 586 / 1783 -> 708 us (4.6 TB/s of the compulsory bytes; a plain 1 GiB copy reaches 5.0),
// FP32 600 -> 363 / 695 -> 479 us; 256^3 FP64 134 -> 80 / 163 -> 101 us, FP32 66 -> 34 / 74 -> 40 us; 128^3
// FP64 22 -> 15 / 23 -> 18 us, FP32 20 -> 12 / 20 -> 14 us; 64^3 FP64 8.3 / 9.3 us; batched, the finest levels
// of 64 instances of 32^3 - 128^3 (45 M cells, FP32): 4 x 75 -> 133 / 146 us.

#include <hip/hip_ext.h>

#include <algorithm>
#include <map>
#include <type_traits>

#include "mg_internal.h"
#include "p2_bodies.h"
#include "sweep_bodies.h"

namespace mgic {

namespace {

constexpr int kHalo = 4;                  // rows on each side: one per half-sweep
constexpr int kMaxThreads = 768;          // 12 waves of up to 168 VGPRs
// a thread's runs in LDS: two buffers of the inputs of four half-sweeps, and one of padding so that 16
// lanes in a row start in different banks
constexpr int kSlots = 9;

// Block b (tiles by planes, rows, z) of a level of n^3 cells, tiles of sh.yr rows x sh.zr runs x sh.cx
// planes.  The last tile of a direction ends at the level's edge and stores only what the tile before it
// does not.  lds: kSlots (sh.yr + 2 kHalo) (sh.zr + 2) runs.  Waves without a run leave at once (a barrier
// waits for the surviving waves only).
template <class T, int MODE>
__device__ __forceinline__ void body_two_sweeps(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ out,
                                                int n, SweepShape sh, T h2, const T* __restrict__ pu,
                                                const T* __restrict__ uold, unsigned b, unsigned nblk, V16<T>* lds) {
    using V = V16<T>;
    constexpr int W = Vec16<T>::W;
    // workgroups go round the 8 XCDs: each XCD takes a contiguous run of tiles, so that the halos of
    // neighbours are in its own L2 (192^3 without: 1.6 times the time)
    b = (b % 8) * (nblk / 8) + min(b % 8, nblk % 8) + b / 8;
    const int NR = sh.zr + 2, ny = sh.yr + 2 * kHalo, cells = ny * NR, cx = sh.cx;
    if ((int)(threadIdx.x & ~63u) >= cells) return;
    const int nzh = n >> 1, nr = nzh / W;
    const int ntz = (nr + sh.zr - 1) / sh.zr, nty = (n + sh.yr - 1) / sh.yr;
    const int zt = (int)(b % (unsigned)ntz), bt = (int)(b / (unsigned)ntz);
    const int yo = (bt % nty) * sh.yr, xo = (bt / nty) * cx, ko = zt * sh.zr;   // first own row, plane, run
    const int y0 = min(yo, n - sh.yr), x0 = min(xo, n - cx), k0 = min(ko, nr - sh.zr);
    auto wrap = [&](int a, int m) { return a < 0 ? a + m : (a >= m ? a - m : a); };
    // idle threads of the last wave shadow the last run (they store nothing)
    const int t = min((int)threadIdx.x, cells - 1);
    const int r = t / NR, k = t - r * NR;
    const bool live = (int)threadIdx.x < cells;
    const bool mine = live && r >= kHalo + (yo - y0) && r < kHalo + sh.yr && k >= 1 + (ko - k0) && k < NR - 1;
    const int y = wrap(y0 + r - kHalo, n);
    const int j0 = wrap((k0 + k - 1) * W, nzh);
    // byte offsets in a plane of the red and the black run; planes start at block-uniform addresses
    const unsigned atr = (unsigned)(y * n + j0) * (unsigned)sizeof(T), atb = atr + (unsigned)nzh * (unsigned)sizeof(T);
    const unsigned np = (unsigned)n * (unsigned)n;
    const int up = (r > 0 ? -NR : 0), dn = (r < ny - 1 ? NR : 0);
    const int lf = (k > 0 ? -1 : 0), rt = (k < NR - 1 ? 1 : 0);
    auto plane = [&](auto* p, int x) { return p + (size_t)((unsigned)wrap(x, n) * np); };
    auto get = [](const T* p, unsigned byte) { return *(const V*)((const char*)p + byte); };
    auto load_start = [&](int x) -> V {              // the half-sweeps' start: the black run (MODE red: the red run)
        if constexpr (MODE == kSweepRed) return get(plane(u, x), atr);
        V v = get(plane(u, x), atb);
        if constexpr (MODE == kSweepCorr) {
            T d[W], o[W];
            corr_delta<T>(pu, uold, nzh, (unsigned)wrap(x, n) >> 1, (unsigned)y >> 1, (unsigned)j0, d);
#pragma unroll
            for (int i = 0; i < W; ++i) o[i] = lane<T>(v, i) + d[i];
            v = pack<T>(o);
        }
        return v;
    };
    auto load_f = [&](int x, unsigned byte) { return get(plane(f, x), byte); };
    // rings of four planes, plane x in slot (x - x0 + 8) & 3 (a constant in the unrolled steps)
    V s0[4], r1[4], b1[4], r2[4], fr[4], fb[4];
    const int first = x0 - 3;                        // plane of the first half-sweep in step 0
    // step s works on p = first + s; slot of plane first + s + d: (s + d) & 3
#pragma unroll
    for (int i = 0; i < 4; ++i) s0[i] = r1[i] = b1[i] = r2[i] = fr[i] = fb[i] = V{};
    s0[3] = load_start(first - 1);
    s0[0] = load_start(first);
    s0[1] = load_start(first + 1);
    fr[0] = load_f(first, atr);
    fb[3] = load_f(first - 1, atb);
    V* own = lds + t * kSlots;
    own[0] = MODE == kSweepRed ? V{} : s0[0];
    own[1] = own[2] = own[3] = V{};
    if constexpr (MODE == kSweepRed) own[1] = r1[3] = s0[3];
    __syncthreads();
    const int steps = cx + 6;
    const V *lup = own + up * kSlots, *ldn = own + dn * kSlots, *lrt = own + rt * kSlots;
    const V* llf = (const V*)((const T*)(own + lf * kSlots) + (W - 1));   // the last entry of the run before
    const unsigned par = (unsigned)(first + 8 + y);   // parity of red cells in plane p: (par + s) & 1
    auto half = [&](int buf, int st, const V& xm, const V& xp, const V& c, const V& fv, bool q) -> V {
        const V ym = lup[buf * 4 + st], yp = ldn[buf * 4 + st];
        const T edge = *(const T*)((q ? lrt : llf) + buf * 4 + st);
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
            nfr = load_f(p + 1, atr);
            nfb = load_f(p, atb);
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
            if (xr >= xo && xr < x0 + cx) *(V*)((char*)plane(out, xr) + atr) = rn;
            if (xb >= xo) *(V*)((char*)plane(out, xb) + atb) = bn;
        }
        if (live) {
            if constexpr (MODE != kSweepRed) own[wr * 4] = s0[ap1];
            own[wr * 4 + 1] = r1[a0];
            own[wr * 4 + 2] = b1[am1];
            own[wr * 4 + 3] = rn;
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

// Tiles of up to kSmallCells runs take their LDS at the launch, so that several blocks share a CU; larger
// ones, one block per CU by their registers, from a fixed array (a launch may ask for 64 KB only, unless
// the function's attribute is raised, which a stream capture would have to come after).
constexpr int kSmallCells = 448, kManyCells = 256;
static_assert(kManyCells <= kSmallCells && kSlots * kSmallCells * 16 <= 65536 && kSlots * kMaxThreads * 16 <= 160 * 1024, "LDS of a block");
extern __shared__ __align__(16) unsigned char sweep_smem[];
template <class V, bool BIG>
__device__ __forceinline__ V* sweep_lds() {
    if constexpr (BIG) {
        __shared__ V big[kSlots * kMaxThreads];
        return big;
    } else {
        return (V*)sweep_smem;
    }
}

template <class T, int MODE, bool BIG>
__global__ void __launch_bounds__(kMaxThreads)
k_two_sweeps(const T* __restrict__ u, const T* __restrict__ f, T* __restrict__ out, int n, SweepShape sh, T h2,
             const T* __restrict__ pu, const T* __restrict__ uold) {
    body_two_sweeps<T, MODE>(u, f, out, n, sh, h2, pu, uold, blockIdx.x, gridDim.x, sweep_lds<V16<T>, BIG>());
}

// the same for the levels of many batched instances: a = {u, f, out, pu, uold}, the tile in C's dims (tiles of
// many levels are small)
template <class T, int MODE>
__global__ void __launch_bounds__(kMaxThreads)
kb_two_sweeps(const BSeg* __restrict__ segs, int nseg, const int* __restrict__ active) {
    unsigned lb;
    const BSeg& s = seg_of(segs, nseg, lb);
    if (!active[s.inst]) return;
    body_two_sweeps<T, MODE>((const T*)s.a[0], (const T*)s.a[1], (T*)s.a[2], s.L.d.x,
                             SweepShape{s.C.d.x, s.C.d.y, s.C.d.z}, (T)(s.h * s.h), (const T*)s.a[3],
                             (const T*)s.a[4], lb, s.nblk, sweep_lds<V16<T>, false>());
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

}  // namespace

int sweep_cells(const SweepShape& s) { return (s.yr + 2 * kHalo) * (s.zr + 2); }

bool two_sweeps_ok(const Lay& L, size_t elem) {
    const int n = L.d.x, W = (int)(16 / elem);
    return L.split && L.d.y == n && L.d.z == n && n >= 16 && n <= 1024 && n % (2 * W) == 0;
}

unsigned sweep_blocks(int n, int W, const SweepShape& s) {
    return (unsigned)cdiv(n, s.yr) * (unsigned)cdiv(n / (2 * W), s.zr) * (unsigned)cdiv(n, s.cx);
}

// The tile for a level of n^3 cells with W cells per run: the least of rounds x steps x time of a step,
// where a CU holds 12 waves (168 VGPRs), a block marches cx + 6 steps, and a step takes 2.2 + the waves per
// SIMD (in 0.36 us; MI355X: 0.77 us with one wave per SIMD, 1.06 with two, 1.5 with three in FP32).  Over
// the shapes of 32^3 .. 256^3 in either precision the choice is within 5 % of the fastest one measured.
// many: the level is one of many in a launch, so the CUs are full and the time per cell counts; blocks of four
// waves and at most 16 planes, three to a CU, leave the launch's end short (64 instances of 32^3 - 128^3, FP32,
// per solve: 9.71 ms; 12 waves 10.56 ms; up to 32 planes 10.00 ms, 8 planes 9.98 ms).  A batch of few instances takes
// the same tiles, which leave CUs idle there, and still gains on half-sweeps: one 256^3 box FP64 5.24 -> 4.71 ms,
// mixed 3.48 -> 2.82; two of 64^3 1.24 -> 1.10 and 1.25 -> 1.10; eight of 32^3 no change.
static SweepShape find_shape(int n, int W, bool many) {
    SweepShape best;
    double least = 1e30;
    const int nr = n / (2 * W);
    for (int tz = 1; tz <= nr && tz <= 32; ++tz) {
        const int zr = cdiv(nr, tz);
        if (cdiv(nr, zr) != tz) continue;
        for (int yr = 8; yr <= 48 && yr <= n; ++yr) {
            const int ty = cdiv(n, yr);
            if (yr > 8 && cdiv(n, yr - 1) == ty) continue;   // the least rows for ty tiles
            const SweepShape tile{yr, zr, 0};
            if (sweep_cells(tile) > (many ? kManyCells : kMaxThreads)) continue;
            const int waves = cdiv(sweep_cells(tile), 64), fit = 12 / waves;
            for (int k = 1; k <= 8; ++k) {                   // k blocks per CU
                int cx = many ? std::min(n, 2 * k) : std::max(4, cdiv(n, std::max(1, 256 * k / (ty * tz))));
                cx = std::min(n, cdiv(n, cdiv(n, cx)));
                const int blocks = ty * tz * cdiv(n, cx), q = cdiv(blocks, 256);
                const int m = many ? fit : std::min(q, fit);
                const double rounds = many ? (double)blocks / m : cdiv(q, fit);
                const double cost = rounds * (cx + 6) * (2.2 + cdiv(m * waves, 4));
                if (cost < least) {
                    least = cost;
                    best = SweepShape{yr, zr, cx};
                }
            }
        }
    }
    return best;
}
// (the search takes up to 20 us of the host's time: kept per thread for the few sizes there are)
SweepShape sweep_shape(int n, int W, bool many) {
    static thread_local std::map<int, SweepShape> found;
    SweepShape& s = found[(n * 8 + W) * 2 + many];
    if (!s.yr) s = find_shape(n, W, many);
    return s;
}

template <class T>
void launch_two_sweeps(const T* u, const T* f, T* out, const Lay& L, double h, int mode, const T* pu, const T* uold,
                             const SweepShape& sh, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
    const int n = L.d.x, cells = sweep_cells(sh);
    const bool big = cells > kSmallCells;
    const unsigned lds = big ? 0u : (unsigned)(kSlots * cells) * 16u;
    const dim3 grid(sweep_blocks(n, Vec16<T>::W, sh)), block((unsigned)cdiv(cells, 64) * 64u);
    const T h2 = (T)(h * h);
    auto run = [&](auto kernel) {
        if (ev0) hipExtLaunchKernelGGL(kernel, grid, block, lds, st, ev0, ev1, 0, u, f, out, n, sh, h2, pu, uold);
        else kernel<<<grid, block, lds, st>>>(u, f, out, n, sh, h2, pu, uold);
    };
    if (mode == kSweepPlain) big ? run(k_two_sweeps<T, kSweepPlain, true>) : run(k_two_sweeps<T, kSweepPlain, false>);
    else if (mode == kSweepCorr) big ? run(k_two_sweeps<T, kSweepCorr, true>) : run(k_two_sweeps<T, kSweepCorr, false>);
    else big ? run(k_two_sweeps<T, kSweepRed, true>) : run(k_two_sweeps<T, kSweepRed, false>);
}

template <class T>
void launch_b_two_sweeps(const BSeg* segs, int nseg, unsigned grid, int cells, const int* active, int mode,
                         hipStream_t st) {
    const unsigned lds = (unsigned)(kSlots * cells) * 16u;
    const dim3 block((unsigned)cdiv(cells, 64) * 64u);
    auto run = [&](auto kernel) { kernel<<<grid, block, lds, st>>>(segs, nseg, active); };
    if (mode == kSweepPlain) run(kb_two_sweeps<T, kSweepPlain>);
    else if (mode == kSweepCorr) run(kb_two_sweeps<T, kSweepCorr>);
    else run(kb_two_sweeps<T, kSweepRed>);
}

template void launch_b_two_sweeps<float>(const BSeg*, int, unsigned, int, const int*, int, hipStream_t);
template void launch_b_two_sweeps<double>(const BSeg*, int, unsigned, int, const int*, int, hipStream_t);
template void launch_two_sweeps<float>(const float*, const float*, float*, const Lay&, double, int, const float*,
                                             const float*, const SweepShape&, hipStream_t, hipEvent_t, hipEvent_t);
template void launch_two_sweeps<double>(const double*, const double*, double*, const Lay&, double, int,
                                              const double*, const double*, const SweepShape&, hipStream_t, hipEvent_t,
                                              hipEvent_t);

}  // namespace mgic
