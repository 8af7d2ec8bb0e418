// Three-dimensional FFTs of real fields for gfx950 and the spectral multipliers of Section 3.5
// (finite-volume and sub-grid deconvolution, the hybrid Poisson correction) and of the real-space
// transfer-function convolution of Section 2.2, fused into the transform's middle pass.
//
// The spectrum of a real field is Hermitian, so only its modes kz = 0 .. M, M = P2 / 2, are formed
// and stored: rows of zs >= M + 1 complex points, half the bytes of a complex transform in every
// pass.  A 3-D transform is three launches of batched 1-D transforms:
//   z  (k_fft_zf / k_fft_zi)  a line of 2M reals is read as M complex points (even, odd), run
//      through a complex transform of length M and separated into M + 1 modes (and back);
//   y, x  (k_fft_lines)  complex lines, strided in memory, transformed in place.
// Between the passes the field stays in one buffer: every workgroup reads all of its lines before
// it writes the same lines back, and at 256^3 that buffer (142 MB) stays in the Infinity Cache.
//
// A workgroup transforms a tile of T threads x 8 points by a Stockham autosort FFT (radix 8, with
// one radix-2 or radix-4 stage when log2 N is not a multiple of 3; Govindaraju et al. 2008, "High
// performance discrete Fourier transforms on graphics processors").  Every thread holds its 8
// points in registers: the first stage takes them straight from global memory and the last stage
// stores them there, so LDS carries only the exchanges between stages (two for N = 256).  The
// stages run small radix first forwards and last backwards: the points that a thread holds after
// the forward transform are those that it needs for the inverse, so the x pass forms the spectrum,
// multiplies it and transforms it back without an exchange, a store or a load in between.
//
// Tiles of the strided passes hold NL lines that are consecutive in kz (8 at N = 256: runs of 128
// bytes).  The lines kz < M of all rows are numbered through, M per row; the Nyquist lines kz = M
// follow after them, so that no tile is left nearly empty for the odd mode.
//
// Bound: the plain passes by the Infinity Cache (a 64 MB device copy reaches 6.9 TB/s), the fused x
// passes by LDS exchanges and FP64 arithmetic at 4-5 waves per SIMD.  Measured at 256^3 (MI355X), per
// field, against the same passes with complex fields through W1, W2, W3 and an LDS round trip per
// stage: z forward 87 -> 58 us, y forward 116 -> 50 us (5.6 TB/s), y inverse 107 -> 45 us, z inverse
// stored 92 (two fields) -> 52 us, table multiplier 193 (two fields) -> 65 us, hybrid correction
// 175 + 164 -> 150 us.  Radix-16 stages (16 points per thread, one exchange at N = 256) measured slower:
// 130-180 VGPRs leave 3 waves per SIMD (y 50 -> 58 us, z inverse 52 -> 65 us).  Holding the hybrid
// kernel to 128 VGPRs spills 72 of them: 150 -> 205 us.

#include "spec_internal.h"

namespace mgic {

namespace {

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }

// radix-4 DFT in registers; forward uses e^{-2 pi i rk/4}, inverse e^{+2 pi i rk/4}
template <bool INV>
__device__ __forceinline__ void dft4(double2& a0, double2& a1, double2& a2, double2& a3) {
    const double2 s02 = cadd(a0, a2), d02 = csub(a0, a2);
    const double2 s13 = cadd(a1, a3), d13 = csub(a1, a3);
    // -i * d13 = (d13.y, -d13.x)
    const double2 mi = INV ? make_double2(-d13.y, d13.x) : make_double2(d13.y, -d13.x);
    a0 = cadd(s02, s13);
    a2 = csub(s02, s13);
    a1 = cadd(d02, mi);
    a3 = csub(d02, mi);
}

// radix-R DFT in registers (R = 2, 4, 8); the radix-8 one is two radix-4 DFTs of the even and odd
// points combined with the eighth roots of unity
template <int R, bool INV>
__device__ __forceinline__ void dft(double2* v) {
    if (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else {
        double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
        double2 o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
        dft4<INV>(e0, e1, e2, e3);
        dft4<INV>(o0, o1, o2, o3);
        const double r2 = 0.70710678118654752440;
        // w^k o_k, w = e^{-i pi / 4} (forward) or e^{+i pi / 4} (inverse)
        const double2 t1 = INV ? make_double2((o1.x - o1.y) * r2, (o1.x + o1.y) * r2)
                               : make_double2((o1.x + o1.y) * r2, (o1.y - o1.x) * r2);
        const double2 t2 = INV ? make_double2(-o2.y, o2.x) : make_double2(o2.y, -o2.x);
        const double2 t3 = INV ? make_double2((-o3.x - o3.y) * r2, (o3.x - o3.y) * r2)
                               : make_double2((o3.y - o3.x) * r2, (-o3.x - o3.y) * r2);
        v[0] = cadd(e0, o0);
        v[4] = csub(e0, o0);
        v[1] = cadd(e1, t1);
        v[5] = csub(e1, t1);
        v[2] = cadd(e2, t2);
        v[6] = csub(e2, t2);
        v[3] = cadd(e3, t3);
        v[7] = csub(e3, t3);
    }
}

// ---- the stages --------------------------------------------------------------------------------
// log2 radix and log2 of the sub-transform length before stage s of a length-2^LGN transform: the
// remainder stage (radix 2^(LGN % 3)) first, or last (REV)
template <int LGN>
struct Stages {
    static constexpr int lgF = LGN % 3;
    static constexpr int count = LGN / 3 + (lgF ? 1 : 0);
    static constexpr int lg_radix(bool rev, int s) {
        if (!lgF) return 3;
        return s == (rev ? count - 1 : 0) ? lgF : 3;
    }
    static constexpr int lg_ns(bool rev, int s) {
        int t = 0;
        for (int i = 0; i < s; ++i) t += lg_radix(rev, i);
        return t;
    }
};

// threads and lines of a strided tile: 8 points per thread; at N = 512 and 1024 twice the threads,
// so that a tile still holds runs of 8 (4) lines
template <int LGN>
constexpr int kFftThreads = LGN >= 9 ? 512 : 256;
template <int LGN>
constexpr int kFftLgLines = (LGN >= 9 ? 12 : 11) - LGN;

// where point i of line l sits in LDS (in complex points), and which line and butterfly item q of a
// stage with P = 2^lgP butterflies per line is.  Strided tiles interleave their lines at an odd
// stride (consecutive lanes are consecutive lines); contiguous ones (LINES = false) keep a line
// together with one point of padding after every 8 (consecutive lanes are consecutive points, and
// a radix-8 stage writes at a stride of 8).
template <int LGN, int LGNL, bool STRIDED>
struct Tile {
    static constexpr int kRow = STRIDED ? (1 << LGNL) + 1 : (1 << LGN) + ((1 << LGN) >> 3);
    static constexpr int kPoints = STRIDED ? (kRow << LGN) : (kRow << LGNL);
    __device__ static __forceinline__ int at(int l, int i) { return STRIDED ? i * kRow + l : l * kRow + i + (i >> 3); }
    __device__ static __forceinline__ void item(int q, int lgP, int& l, int& j) {
        if (STRIDED) {
            l = q & ((1 << LGNL) - 1);
            j = q >> LGNL;
        } else {
            l = q >> lgP;
            j = q & ((1 << lgP) - 1);
        }
    }
};

// Stage S on the thread's 8 points (8 / R butterflies): twiddle point r of butterfly j by
// w^(r k N / (Ns R)), k = j mod Ns, then the radix-R DFT.  twl holds e^{-2 pi i t / N} in LDS.
template <int LGN, int LGNL, bool STRIDED, bool REV, bool INV, int S, int T>
__device__ __forceinline__ void stage_dft(double2* v, const double2* twl) {
    constexpr int lgR = Stages<LGN>::lg_radix(REV, S), R = 1 << lgR, lgNs = Stages<LGN>::lg_ns(REV, S);
#pragma unroll
    for (int it = 0; it < 8 / R; ++it) {
        if (lgNs > 0) {
            int l, j;
            Tile<LGN, LGNL, STRIDED>::item((int)threadIdx.x + it * T, LGN - lgR, l, j);
            const int step = (j & ((1 << lgNs) - 1)) << (LGN - lgNs - lgR);
#pragma unroll
            for (int r = 1; r < R; ++r) {
                double2 w = twl[r * step];
                if (INV) w.y = -w.y;
                v[it * R + r] = cmul(v[it * R + r], w);
            }
        }
        dft<R, INV>(v + it * R);
    }
}

// point r of butterfly j before stage S, and where the stage's DFT puts it
template <int LGN, bool REV, int S>
__device__ __forceinline__ int point_in(int j, int r) {
    return j + (r << (LGN - Stages<LGN>::lg_radix(REV, S)));
}
template <int LGN, bool REV, int S>
__device__ __forceinline__ int point_out(int j, int r) {
    constexpr int lgR = Stages<LGN>::lg_radix(REV, S), lgNs = Stages<LGN>::lg_ns(REV, S);
    const int k = j & ((1 << lgNs) - 1);
    return ((j - k) << lgR) + k + (r << lgNs);
}

// calls f(slot, line, point) for the 8 points that the thread holds before (OUT: after) stage S
template <int LGN, int LGNL, bool STRIDED, bool REV, int S, bool OUT, int T, typename F>
__device__ __forceinline__ void each_point(F&& f) {
    constexpr int lgR = Stages<LGN>::lg_radix(REV, S), R = 1 << lgR;
#pragma unroll
    for (int it = 0; it < 8 / R; ++it) {
        int l, j;
        Tile<LGN, LGNL, STRIDED>::item((int)threadIdx.x + it * T, LGN - lgR, l, j);
#pragma unroll
        for (int r = 0; r < R; ++r)
            f(it * R + r, l, OUT ? point_out<LGN, REV, S>(j, r) : point_in<LGN, REV, S>(j, r));
    }
}

// exchange through LDS: the points after stage S become those before stage S + 1
template <int LGN, int LGNL, bool STRIDED, bool REV, int S, int T>
__device__ __forceinline__ void exchange(double2* v, double2* lds) {
    __syncthreads();   // the previous use of lds is over
    each_point<LGN, LGNL, STRIDED, REV, S, true, T>(
        [&](int s, int l, int i) { lds[Tile<LGN, LGNL, STRIDED>::at(l, i)] = v[s]; });
    __syncthreads();
    each_point<LGN, LGNL, STRIDED, REV, S + 1, false, T>(
        [&](int s, int l, int i) { v[s] = lds[Tile<LGN, LGNL, STRIDED>::at(l, i)]; });
}

// the whole transform of the 8 points in v: before, those of stage 0; after, those of the last stage
template <int LGN, int LGNL, bool STRIDED, bool INV, int T, int S = 0>
__device__ __forceinline__ void fft_regs(double2* v, double2* lds, const double2* twl) {
    if constexpr (S < Stages<LGN>::count) {
        stage_dft<LGN, LGNL, STRIDED, INV, INV, S, T>(v, twl);
        if constexpr (S + 1 < Stages<LGN>::count) {
            exchange<LGN, LGNL, STRIDED, INV, S, T>(v, lds);
            fft_regs<LGN, LGNL, STRIDED, INV, T, S + 1>(v, lds, twl);
        }
    }
}

// ---- multipliers -------------------------------------------------------------------------------
// the multiplier of spectral element (kx, ky, kz) = (i, a, b), b <= P2 / 2, applied to v
template <int SYM>
__device__ __forceinline__ double2 apply_sym(const FftPass& A, int i, int a, int b, double2 v) {
    const double c = A.sym_scale;
    if (SYM == kSymSeparable) {
        const double m = ((A.tab_x[i] * A.tab_y[a]) * A.tab_z[b]) * c;
        return make_double2(v.x * m, v.y * m);
    }
    if (SYM == kSymTable) {
        const double m = A.tab[(long long)i * A.tab_si + (long long)a * A.tab_sa + b] * c;
        return make_double2(v.x * m, v.y * m);
    }
    if (SYM == kSymInvLap) {
        // 1 / lambda(k), lambda = sum_axes of the per-axis Laplacian symbol; the k = 0 mode -> 0
        const double lam = (A.tab_x[i] + A.tab_y[a]) + A.tab_z[b];
        if (i == 0 && a == 0 && b == 0) return make_double2(0.0, 0.0);
        const double m = c / lam;
        return make_double2(v.x * m, v.y * m);
    }
    // kSymReplace: modes below the coarse grid's Nyquist on every axis take 8 C(m) prod_a
    // e^{-i pi m_a / P_a} (per-axis phase tables hold cos, sin pairs); the rest keep the fine spectrum
    const int px = A.sym_n[0], py = A.sym_n[1];
    const int mx = i < px / 2 ? i : i - px, my = a < py / 2 ? a : a - py;
    const int cx = A.cn[0], cy = A.cn[1], cz = A.cn[2];
    if (2 * abs(mx) < cx && 2 * abs(my) < cy && 2 * b < cz) {
        const int ix = mx < 0 ? mx + cx : mx, iy = my < 0 ? my + cy : my;
        const double2 C = A.csp[((long long)ix * cy + iy) * A.csp_zs + b];
        double2 w = make_double2(8.0 * C.x, 8.0 * C.y);
        w = cmul(w, make_double2(A.tab_x[2 * i], A.tab_x[2 * i + 1]));
        w = cmul(w, make_double2(A.tab_y[2 * a], A.tab_y[2 * a + 1]));
        w = cmul(w, make_double2(A.tab_z[2 * b], A.tab_z[2 * b + 1]));
        return make_double2(w.x * c, w.y * c);
    }
    return make_double2(v.x * A.fine_scale, v.y * A.fine_scale);
}

// ---- strided passes ----------------------------------------------------------------------------
// The lines of a pass: kz < M of every row a < na, M per row, then kz = M of every row.
__device__ __forceinline__ bool line_at(const FftPass& A, long long L, int& a, int& b) {
    const long long reg = (long long)A.na << A.lgM;
    if (L < reg) {
        a = (int)(L >> A.lgM);
        b = (int)(L & ((1 << A.lgM) - 1));
        return true;
    }
    a = (int)(L - reg);
    b = 1 << A.lgM;
    return a < A.na;
}

// One pass over lines of length N = 2^LGN, field blockIdx.y.  OP: kFftForward, kFftInverse; kFftRe
// forward with the real part stored into a table; kFftFwdSymInv forward, multiply, inverse in one
// launch; kFftHybrid the same with the three components of the hybrid correction, from one input
// into fields 0, 1, 2 (the spectrum stays in registers between them); kFftHybridOne with one of them, into a
// field of its own.
template <int LGN, int OP, int SYM>
__global__ __launch_bounds__(kFftThreads<LGN>) void k_fft_lines(FftPass A) {
    constexpr int T = kFftThreads<LGN>, LGNL = kFftLgLines<LGN>, NL = 1 << LGNL, N = 1 << LGN;
    constexpr bool kInv = OP == kFftInverse;
    using TL = Tile<LGN, LGNL, true>;
    extern __shared__ __align__(16) unsigned char fft_smem[];
    double2* lds = (double2*)fft_smem;
    double2* twl = lds + TL::kPoints;
    const double2* in = (const double2*)A.in + (long long)blockIdx.y * A.fs;
    double2* out = (double2*)A.out + (long long)blockIdx.y * A.fs;
    // the lines of this thread's points: one (NL <= T), or one per butterfly
    constexpr int kL = NL > T ? NL / T : 1;
    int la[kL], lb[kL];
    bool ok[kL];
#pragma unroll
    for (int t = 0; t < kL; ++t)
        ok[t] = line_at(A, ((long long)blockIdx.x << LGNL) + (((int)threadIdx.x + t * T) & (NL - 1)), la[t], lb[t]);
    auto slot_line = [](int s) { return kL == 1 ? 0 : s >> LGN; };   // kL > 1: one butterfly a line
    double2 v[8];
    each_point<LGN, LGNL, true, kInv, 0, false, T>([&](int s, int l, int i) {
        const int t = slot_line(s);
        v[s] = make_double2(0.0, 0.0);
        if (ok[t] && i >= A.in_lo && i < A.in_hi)
            v[s] = in[(long long)la[t] * A.in_sa + lb[t] + (long long)i * A.in_si];
    });
    for (int t = (int)threadIdx.x; t < N; t += T) twl[t] = A.tw[t << (A.lgtw - LGN)];
    constexpr int kLast = Stages<LGN>::count - 1;
    auto store = [&](double2* to) {
        each_point<LGN, LGNL, true, true, kLast, true, T>([&](int s, int l, int i) {
            const int t = slot_line(s);
            if (ok[t] && i >= A.out_lo && i < A.out_hi)
                to[(long long)la[t] * A.out_sa + lb[t] + (long long)i * A.out_si] = v[s];
        });
    };
    if constexpr (kInv) {
        fft_regs<LGN, LGNL, true, true, T>(v, lds, twl);
        store(out);
    } else {
        fft_regs<LGN, LGNL, true, false, T>(v, lds, twl);
        if constexpr (OP == kFftForward || OP == kFftRe) {
            each_point<LGN, LGNL, true, false, kLast, true, T>([&](int s, int l, int i) {
                const int t = slot_line(s);
                if (!ok[t] || i >= A.out_hi) return;
                const long long at = (long long)la[t] * A.out_sa + lb[t] + (long long)i * A.out_si;
                if (OP == kFftRe) ((double*)A.out)[at] = v[s].x;
                else out[at] = v[s];
            });
        } else if constexpr (OP == kFftFwdSymInv) {
            each_point<LGN, LGNL, true, false, kLast, true, T>([&](int s, int l, int i) {
                const int t = slot_line(s);
                if (ok[t]) v[s] = apply_sym<SYM>(A, i, la[t], lb[t], v[s]);
            });
            fft_regs<LGN, LGNL, true, true, T>(v, lds, twl);
            store(out);
        } else {
            // hybrid correction, component c: i s_c f~, s_c = -k_c / k^2 - g_c / lambda; per-axis
            // blocks [k^2 | lambda_1d | k (0 on Nyquist) | g (0 on Nyquist)]
            const int px = A.sym_n[0], py = A.sym_n[1], pz = A.sym_n[2];
            double2 f[8];
            double rk[8], rl[8];   // -scale / k^2 and -scale / lambda, shared by the components
            each_point<LGN, LGNL, true, false, kLast, true, T>([&](int s, int l, int i) {
                const int t = slot_line(s);
                f[s] = v[s];
                rk[s] = rl[s] = 0.0;
                if (!ok[t]) return;
                const double k2 = (A.tab_x[i] + A.tab_y[la[t]]) + A.tab_z[lb[t]];
                if (k2 == 0.0) return;
                rk[s] = -A.sym_scale / k2;
                rl[s] = -A.sym_scale / ((A.tab_x[px + i] + A.tab_y[py + la[t]]) + A.tab_z[pz + lb[t]]);
            });
            constexpr int kComps = OP == kFftHybrid ? 3 : 1;
#pragma unroll
            for (int k = 0; k < kComps; ++k) {
                const int c = kComps == 3 ? k : A.comp;
                each_point<LGN, LGNL, true, false, kLast, true, T>([&](int s, int l, int i) {
                    const int t = slot_line(s);
                    if (!ok[t]) return;
                    const int a = la[t], b = lb[t];
                    const double kc = c == 0 ? A.tab_x[2 * px + i] : (c == 1 ? A.tab_y[2 * py + a] : A.tab_z[2 * pz + b]);
                    const double gc = c == 0 ? A.tab_x[3 * px + i] : (c == 1 ? A.tab_y[3 * py + a] : A.tab_z[3 * pz + b]);
                    const double m = kc * rk[s] + gc * rl[s];
                    v[s] = make_double2(-f[s].y * m, f[s].x * m);
                });
                fft_regs<LGN, LGNL, true, true, T>(v, lds, twl);
                store((double2*)A.out + (long long)k * A.fs);
            }
        }
    }
}

// ---- z passes ----------------------------------------------------------------------------------
constexpr int kZThreads = 256;
template <int LGM>
constexpr int kZLgLines = 11 - LGM;

// line L is row y = L % rows of x plane L / rows, counted from the first row of the pass
struct ZLine {
    int x, y;
    __device__ __forceinline__ ZLine(const FftPass& A, int L) {
        x = (int)((unsigned)L / (unsigned)A.rows);
        y = L - x * A.rows;
    }
    __device__ __forceinline__ long long spectrum(const FftPass& A) const { return ((long long)x * A.plane + y) * A.zs; }
    __device__ __forceinline__ long long real(const FftPass& A) const { return x * A.rsx + y * A.rsy; }
};

// points z, z + 1 of the input of a multi-scale convolution on a patch's padded domain D' (the
// patch at [n/2, 3n/2) of it), formed from the noise mu and its parent's par:
//   kPrepSelf   the noise inside the patch, noise minus its parent's value on the padding
//   kPrepBnd    0 inside the patch, noise minus its parent's value on the padding
//   kPrepOpen   the noise, 0 in the cells that the next patch covers
__device__ __forceinline__ double2 conv_input(const ConvPrep& C, int x, int y, int z, double2 m) {
    if (C.mode == kPrepOpen) {
        if (x >= C.lo[0] && x < C.hi[0] && y >= C.lo[1] && y < C.hi[1]) {
            if (z >= C.lo[2] && z < C.hi[2]) m.x = 0.0;
            if (z + 1 >= C.lo[2] && z + 1 < C.hi[2]) m.y = 0.0;
        }
        return m;
    }
    // the patch's bounds are even along z: both points lie inside, or both outside
    if (x >= C.lo[0] && x < C.hi[0] && y >= C.lo[1] && y < C.hi[1] && z >= C.lo[2] && z < C.hi[2])
        return C.mode == kPrepSelf ? m : make_double2(0.0, 0.0);
    int p[3] = {C.pb.lo[0] + (x >> 1), C.pb.lo[1] + (y >> 1), C.pb.lo[2] + (z >> 1)};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (C.pb.wrap) {   // D' covers at most the whole base: one turn is enough
            if (p[a] < 0) p[a] += C.pb.wrap;
            if (p[a] >= C.pb.wrap) p[a] -= C.pb.wrap;
        }
        p[a] += C.pb.po[a];
    }
    const double v = C.par[((long long)p[0] * C.pb.pd[1] + p[1]) * C.pb.pd[2] + p[2]];
    return make_double2(m.x - v, m.y - v);
}

// Forward z pass: the reals in_lo <= z < in_hi of every line, zero-extended to N = 2M = 2^(LGM + 1),
// to modes 0 .. M.  PREP: the reals are formed by conv_input.
// With Z the transform of the complex line (x_2i + i x_2i+1), E = (Z[k] + conj Z[M-k]) / 2 and
// O = (Z[k] - conj Z[M-k]) / 2:  X[k] = E - i w^k O and X[M-k] = conj(E + i w^k O), w = e^{-2 pi i / N}.
template <int LGM, bool PREP>
__global__ __launch_bounds__(kZThreads) void k_fft_zf(FftPass A, ConvPrep C) {
    constexpr int T = kZThreads, LGNL = kZLgLines<LGM>, M = 1 << LGM;
    using TL = Tile<LGM, LGNL, false>;
    extern __shared__ __align__(16) unsigned char fft_smem[];
    double2* lds = (double2*)fft_smem;
    double2* twl = lds + TL::kPoints;
    const double* in = (const double*)A.rin[blockIdx.y];
    double2* out = (double2*)A.out + (long long)blockIdx.y * A.fs;
    const int L0 = (int)blockIdx.x << LGNL;
    const bool pairs = A.vec & (1 << blockIdx.y);
    double2 v[8];
    auto load = [&](int s, int l, int i) {
        const int L = L0 + l, z = 2 * i;
        v[s] = make_double2(0.0, 0.0);
        if (L < A.na && z >= A.in_lo && z < A.in_hi) {
            const ZLine zl(A, L);
            const double* p = in + zl.real(A) + (z - A.in_lo);
            if (pairs) {
                v[s] = *(const double2*)p;
            } else {
                v[s].x = p[0];
                if (z + 1 < A.in_hi) v[s].y = p[1];
            }
            if (PREP) v[s] = conv_input(C, zl.x + C.x0, zl.y + C.y0, z, v[s]);
        }
    };
    if constexpr (LGM == 0) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int l = (int)threadIdx.x + s * T, L = L0 + l;
            load(s, l, 0);
            if (L < A.na) {
                const long long at = ZLine(A, L).spectrum(A);
                out[at] = make_double2(v[s].x + v[s].y, 0.0);
                out[at + 1] = make_double2(v[s].x - v[s].y, 0.0);
            }
        }
    } else {
        each_point<LGM, LGNL, false, false, 0, false, T>(load);
        for (int t = (int)threadIdx.x; t < M; t += T) twl[t] = A.tw[t << (A.lgtw - LGM)];
        fft_regs<LGM, LGNL, false, false, T>(v, lds, twl);
        __syncthreads();
        each_point<LGM, LGNL, false, false, Stages<LGM>::count - 1, true, T>(
            [&](int s, int l, int i) { lds[TL::at(l, i)] = v[s]; });
        __syncthreads();
        constexpr int kItems = 1 << (LGM - 1 + LGNL);
#pragma unroll
        for (int q = (int)threadIdx.x; q < kItems; q += T) {
            const int l = q >> (LGM - 1), k = q & (M / 2 - 1), L = L0 + l;
            if (L >= A.na) continue;
            double2* row = out + ZLine(A, L).spectrum(A);
            const double2 a = lds[TL::at(l, k)];
            if (k == 0) {
                row[0] = make_double2(a.x + a.y, 0.0);
                row[M] = make_double2(a.x - a.y, 0.0);
                const double2 h = lds[TL::at(l, M / 2)];
                row[M / 2] = make_double2(h.x, -h.y);
                continue;
            }
            const double2 b = lds[TL::at(l, M - k)];
            const double2 E = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));
            const double2 O = make_double2(0.5 * (a.x - b.x), 0.5 * (a.y + b.y));
            const double2 w = A.tw[k << (A.lgtw - LGM - 1)];
            const double2 wo = cmul(w, O);
            const double2 t = make_double2(wo.y, -wo.x);   // -i w O
            row[k] = cadd(E, t);
            row[M - k] = make_double2(E.x - t.x, t.y - E.y);
        }
    }
}

// Inverse z pass: modes 0 .. M to the reals out_lo <= z < out_hi of every line, stored or added.
// 2 Z[k] = E + O and 2 Z[M-k] = conj(E - O), E = X[k] + conj X[M-k], O = i conj(w^k) (X[k] - conj X[M-k]).
template <int LGM, bool ADD>
__global__ __launch_bounds__(kZThreads) void k_fft_zi(FftPass A) {
    constexpr int T = kZThreads, LGNL = kZLgLines<LGM>, M = 1 << LGM;
    using TL = Tile<LGM, LGNL, false>;
    extern __shared__ __align__(16) unsigned char fft_smem[];
    double2* lds = (double2*)fft_smem;
    double2* twl = lds + TL::kPoints;
    const double2* in = (const double2*)A.in + (long long)blockIdx.y * A.fs;
    double* out = (double*)A.rout[blockIdx.y];
    const int L0 = (int)blockIdx.x << LGNL;
    const bool pairs = A.vec & (1 << blockIdx.y);
    double2 v[8];
    auto store = [&](int s, int l, int i) {
        const int L = L0 + l, z = 2 * i - A.out_lo;
        const int m = A.out_hi - A.out_lo;
        if (L >= A.na || z < 0 || z >= m) return;
        double* p = out + ZLine(A, L).real(A) + z;
        if (pairs) {
            double2 o = v[s];
            if (ADD) o = cadd(*(const double2*)p, o);
            *(double2*)p = o;
        } else {
            p[0] = ADD ? p[0] + v[s].x : v[s].x;
            if (z + 1 < m) p[1] = ADD ? p[1] + v[s].y : v[s].y;
        }
    };
    if constexpr (LGM == 0) {
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int l = (int)threadIdx.x + s * T, L = L0 + l;
            if (L < A.na) {
                const long long at = ZLine(A, L).spectrum(A);
                const double2 x0 = in[at], x1 = in[at + 1];
                v[s] = make_double2(x0.x + x1.x, x0.x - x1.x);
                store(s, l, 0);
            }
        }
    } else {
        constexpr int kItems = 1 << (LGM - 1 + LGNL);
        constexpr int kPer = kItems / T;
        double2 x[kPer], y[kPer], xh[kPer];
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            const int q = (int)threadIdx.x + n * T;
            const int l = q >> (LGM - 1), k = q & (M / 2 - 1), L = L0 + l;
            x[n] = y[n] = xh[n] = make_double2(0.0, 0.0);
            if (L < A.na) {
                const double2* row = in + ZLine(A, L).spectrum(A);
                x[n] = row[k];
                y[n] = row[M - k];
                if (k == 0) xh[n] = row[M / 2];
            }
        }
        for (int t = (int)threadIdx.x; t < M; t += T) twl[t] = A.tw[t << (A.lgtw - LGM)];
#pragma unroll
        for (int n = 0; n < kPer; ++n) {
            const int q = (int)threadIdx.x + n * T;
            const int l = q >> (LGM - 1), k = q & (M / 2 - 1);
            if (k == 0) {
                lds[TL::at(l, 0)] = make_double2(x[n].x + y[n].x, x[n].x - y[n].x);
                lds[TL::at(l, M / 2)] = make_double2(2.0 * xh[n].x, -2.0 * xh[n].y);
            } else {
                const double2 E = make_double2(x[n].x + y[n].x, x[n].y - y[n].y);
                const double2 D = make_double2(x[n].x - y[n].x, x[n].y + y[n].y);
                const double2 w = A.tw[k << (A.lgtw - LGM - 1)];
                const double2 wd = cmul(make_double2(w.x, -w.y), D);
                const double2 O = make_double2(-wd.y, wd.x);   // i conj(w) D
                lds[TL::at(l, k)] = cadd(E, O);
                lds[TL::at(l, M - k)] = make_double2(E.x - O.x, O.y - E.y);
            }
        }
        __syncthreads();
        each_point<LGM, LGNL, false, true, 0, false, T>(
            [&](int s, int l, int i) { v[s] = lds[TL::at(l, i)]; });
        fft_regs<LGM, LGNL, false, true, T>(v, lds, twl);
        each_point<LGM, LGNL, false, true, Stages<LGM>::count - 1, true, T>(store);
    }
}

// Per-axis multiplier tables.  Mode m of an axis of P points (m = t for t < P/2, t - P above) has
// kh = 2 pi m / P.  kind kSymFv: 1 / sinc(kh/2); kSymSg: 1 / cos(kh/4); hybrid: the four blocks
// [kh^2 | Laplacian symbol of the order | kh, 0 on Nyquist | gradient symbol g, 0 on Nyquist].
// kind 0: none.  The first 2^lg threads write the twiddles e^{-2 pi i t / 2^lg}.
__global__ void k_spec_tables(double2* tw, int lg, double* t0, double* t1, double* t2, int p0, int p1, int p2,
                              int kind, int lap_order, int grad_order) {
    int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (t < (1 << lg)) {
        double s, c;
        sincospi(2.0 * (double)t / (double)(1 << lg), &s, &c);
        tw[t] = make_double2(c, -s);
        return;
    }
    t -= 1 << lg;
    if (kind == 0) return;
    double* tab;
    int P;
    if (t < p0) {
        tab = t0;
        P = p0;
    } else if (t < p0 + p1) {
        tab = t1;
        P = p1;
        t -= p0;
    } else if (t < p0 + p1 + p2) {
        tab = t2;
        P = p2;
        t -= p0 + p1;
    } else {
        return;
    }
    const int m = t < P / 2 ? t : t - P;
    const double q = 2.0 * (double)m / (double)P;   // kh / pi
    const double kh = 3.14159265358979323846 * q;
    if (kind == kSpecFv) {
        double s, c;
        sincospi(0.5 * q, &s, &c);
        tab[t] = m == 0 ? 1.0 : (0.5 * kh) / s;
        return;
    }
    if (kind == kSpecSg) {
        tab[t] = 1.0 / cospi(0.25 * q);
        return;
    }
    if (kind == kSpecPoisson) {   // the 1-D Laplacian symbol of the order, in grid units
        double s1, c1, s2, c2, s3, c3;
        sincospi(q, &s1, &c1);
        sincospi(2.0 * q, &s2, &c2);
        sincospi(3.0 * q, &s3, &c3);
        if (lap_order == 2) tab[t] = -2.0 * (1.0 - c1);
        else if (lap_order == 4) tab[t] = -(c2 - 16.0 * c1 + 15.0) / 6.0;
        else tab[t] = -(-2.0 * c3 + 27.0 * c2 - 270.0 * c1 + 245.0) / 90.0;
        return;
    }
    if (kind == kSpecReplace) {   // e^{-i pi m / P}: the fine centres sit a quarter coarse cell off
        double s, c;
        sincospi((double)m / (double)P, &s, &c);
        tab[2 * t] = c;
        tab[2 * t + 1] = -s;
        return;
    }
    double s1, c1, s2, c2, s3, c3;
    sincospi(q, &s1, &c1);
    sincospi(2.0 * q, &s2, &c2);
    sincospi(3.0 * q, &s3, &c3);
    double lam;
    if (lap_order == 2) lam = -2.0 * (1.0 - c1);
    else if (lap_order == 4) lam = -(c2 - 16.0 * c1 + 15.0) / 6.0;
    else lam = -(-2.0 * c3 + 27.0 * c2 - 270.0 * c1 + 245.0) / 90.0;
    double g;
    if (grad_order == 4) g = (8.0 * s1 - s2) / 6.0;
    else g = (45.0 * s1 - 9.0 * s2 + s3) / 30.0;
    const bool nyq = 2 * t == P;
    tab[t] = kh * kh;
    tab[P + t] = lam;
    tab[2 * P + t] = nyq ? 0.0 : kh;
    tab[3 * P + t] = nyq ? 0.0 : g;
}


// ---- launches ----------------------------------------------------------------------------------
hipError_t raise_lds(const void* fn, unsigned lds) {
    if (lds <= 65536u) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

template <int LGN, int OP, int SYM>
hipError_t run_lines(const FftPass& A, hipStream_t st) {
    constexpr int LGNL = kFftLgLines<LGN>;
    const unsigned lds = (unsigned)((Tile<LGN, LGNL, true>::kPoints + (1 << LGN)) * sizeof(double2));
    const hipError_t e = raise_lds((const void*)k_fft_lines<LGN, OP, SYM>, lds);
    if (e != hipSuccess) return e;
    const long long lines = ((long long)A.na << A.lgM) + A.na;
    const unsigned blocks = (unsigned)((lines + (1 << LGNL) - 1) >> LGNL);
    if (blocks == 0) return hipSuccess;
    k_fft_lines<LGN, OP, SYM><<<dim3(blocks, (unsigned)A.nf), kFftThreads<LGN>, lds, st>>>(A);
    return hipGetLastError();
}

// DIR 0: forward, 1: inverse stored, 2: inverse added, 3: forward of a convolution's input
template <int LGM, int DIR>
hipError_t run_z(const FftPass& A, const ConvPrep& C, hipStream_t st) {
    constexpr int LGNL = kZLgLines<LGM>;
    const unsigned lds = (unsigned)((Tile<LGM, LGNL, false>::kPoints + (1 << LGM)) * sizeof(double2));
    const unsigned blocks = (unsigned)(((long long)A.na + (1 << LGNL) - 1) >> LGNL);
    if (blocks == 0) return hipSuccess;
    const dim3 grid(blocks, (unsigned)A.nf);
    if constexpr (DIR == 0) k_fft_zf<LGM, false><<<grid, kZThreads, lds, st>>>(A, C);
    else if constexpr (DIR == 1) k_fft_zi<LGM, false><<<grid, kZThreads, lds, st>>>(A);
    else if constexpr (DIR == 2) k_fft_zi<LGM, true><<<grid, kZThreads, lds, st>>>(A);
    else k_fft_zf<LGM, true><<<grid, kZThreads, lds, st>>>(A, C);
    return hipGetLastError();
}

template <int OP, int SYM>
hipError_t lines_of_length(const FftPass& A, hipStream_t st) {
    switch (A.lgN) {
        case 1: return run_lines<1, OP, SYM>(A, st);
        case 2: return run_lines<2, OP, SYM>(A, st);
        case 3: return run_lines<3, OP, SYM>(A, st);
        case 4: return run_lines<4, OP, SYM>(A, st);
        case 5: return run_lines<5, OP, SYM>(A, st);
        case 6: return run_lines<6, OP, SYM>(A, st);
        case 7: return run_lines<7, OP, SYM>(A, st);
        case 8: return run_lines<8, OP, SYM>(A, st);
        case 9: return run_lines<9, OP, SYM>(A, st);
        case 10: return run_lines<10, OP, SYM>(A, st);
        default: return hipErrorInvalidValue;
    }
}

template <int DIR>
hipError_t z_of_length(const FftPass& A, const ConvPrep& C, hipStream_t st) {
    switch (A.lgM) {
        case 0: return run_z<0, DIR>(A, C, st);
        case 1: return run_z<1, DIR>(A, C, st);
        case 2: return run_z<2, DIR>(A, C, st);
        case 3: return run_z<3, DIR>(A, C, st);
        case 4: return run_z<4, DIR>(A, C, st);
        case 5: return run_z<5, DIR>(A, C, st);
        case 6: return run_z<6, DIR>(A, C, st);
        case 7: return run_z<7, DIR>(A, C, st);
        case 8: return run_z<8, DIR>(A, C, st);
        case 9: return run_z<9, DIR>(A, C, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_spec_tables(double2* tw, int lg, double* t0, double* t1, double* t2, const int P[3], int kind,
                              int lap_order, int grad_order, hipStream_t st) {
    const int total = (1 << lg) + (kind ? P[0] + P[1] + P[2] : 0);
    k_spec_tables<<<(total + kBlock - 1) / kBlock, kBlock, 0, st>>>(tw, lg, t0, t1, t2, P[0], P[1], P[2], kind,
                                                                     lap_order, grad_order);
    return hipGetLastError();
}

hipError_t launch_fft_z_forward(const FftPass& A, const ConvPrep* prep, hipStream_t st) {
    return prep ? z_of_length<3>(A, *prep, st) : z_of_length<0>(A, ConvPrep(), st);
}

hipError_t launch_fft_z_inverse(const FftPass& A, bool add, hipStream_t st) {
    return add ? z_of_length<2>(A, ConvPrep(), st) : z_of_length<1>(A, ConvPrep(), st);
}

hipError_t launch_fft_lines(const FftPass& A, int op, int sym, hipStream_t st) {
    if (op == kFftForward) return lines_of_length<kFftForward, 0>(A, st);
    if (op == kFftInverse) return lines_of_length<kFftInverse, 0>(A, st);
    if (op == kFftRe) return lines_of_length<kFftRe, 0>(A, st);
    if (op == kFftHybrid) return lines_of_length<kFftHybrid, 0>(A, st);
    if (op == kFftHybridOne) return lines_of_length<kFftHybridOne, 0>(A, st);
    if (op != kFftFwdSymInv) return hipErrorInvalidValue;
    switch (sym) {
        case kSymSeparable: return lines_of_length<kFftFwdSymInv, kSymSeparable>(A, st);
        case kSymTable: return lines_of_length<kFftFwdSymInv, kSymTable>(A, st);
        case kSymReplace: return lines_of_length<kFftFwdSymInv, kSymReplace>(A, st);
        case kSymInvLap: return lines_of_length<kFftFwdSymInv, kSymInvLap>(A, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mgic
