// Host side of the spectral operations (Section 3.5 of Hahn & Abel 2011): the finite-volume and
// sub-grid deconvolutions and the hybrid Poisson correction on the finest grid, built on the
// three-pass FFT of k_fft.hip.
//
// Pipeline for a real field f of n0 x n1 x n2 cells transformed on P0 x P1 x P2 points (P = n on
// periodic grids, the zero-padded isolated length otherwise), z contiguous; the spectrum of a real
// field is Hermitian, so W holds its modes kz = 0 .. P2 / 2 only, in rows of zs points:
//   z pass   f -> W [n0][n1 of P1][zs]   (lines zero-extended from n2 to P2)
//   y pass   W in place                  (n1 rows zero-extended to P1)
//   x pass   W in place: forward, multiplier, inverse   (one launch)
//   y pass   W in place, inverse
//   z pass   W (inverse) -> real output [n0][n1][n2]
// Only the first n points of x and z are ever stored: lines that are zero by padding are not
// transformed, and output points outside the patch are not computed past the axis they lie on.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>

#include "spec_internal.h"
#include "mgic.h"

namespace mgic {

namespace {

#define SP_HIP(call)                                                                             \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess) {                                                                  \
            (void)hipGetLastError();                                                             \
            return report_error(MG_EHIP, (std::string(#call) + ": " + hipGetErrorString(e_)).c_str()); \
        }                                                                                        \
    } while (0)

int pad_len(int n) {
    int p = 1;
    while (p < 2 * n) p *= 2;
    return p;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

FftPass pass_base(const SpecGrid& S, int axis, int nf) {
    FftPass A;
    A.lgN = S.lg[axis];
    A.lgM = S.lg[2] - 1;
    A.lgtw = S.lgtw;
    A.tw = S.tw;
    A.nf = nf;
    A.zs = S.zs;
    A.fs = (long long)S.field();
    A.in = S.W;
    A.out = S.W;
    return A;
}

// x planes lo0 <= x < hi0 of the field
FftPass pass_y(const SpecGrid& S, const SpecField& f, int nf) {
    FftPass A = pass_base(S, 1, nf);
    A.na = f.hi[0] - f.lo[0];
    A.in_sa = A.out_sa = (long long)S.P[1] * S.zs;
    A.in_si = A.out_si = S.zs;
    A.in = A.out = S.W + (long long)f.lo[0] * S.P[1] * S.zs;
    return A;
}

FftPass pass_x(const SpecGrid& S) {
    FftPass A = pass_base(S, 0, 1);
    A.na = S.P[1];
    A.in_sa = A.out_sa = S.zs;
    A.in_si = A.out_si = (long long)S.P[1] * S.zs;
    A.tab_x = S.tab[0];
    A.tab_y = S.tab[1];
    A.tab_z = S.tab[2];
    for (int a = 0; a < 3; ++a) A.sym_n[a] = S.P[a];
    return A;
}

FftPass pass_z(const SpecGrid& S, const SpecField& f, int nf) {
    FftPass A = pass_base(S, 2, nf);
    A.rows = f.hi[1] - f.lo[1];
    A.na = (f.hi[0] - f.lo[0]) * A.rows;
    A.plane = S.P[1];
    A.rsx = f.sx;
    A.rsy = f.sy;
    A.in = A.out = S.W + ((long long)f.lo[0] * S.P[1] + f.lo[1]) * S.zs;
    return A;
}

// whether the real lines of a field can be read and written as 16-byte pairs of points
bool by_pairs(const SpecField& f, const double* p) {
    return f.sx % 2 == 0 && f.sy % 2 == 0 && f.hi[2] % 2 == 0 && (((uintptr_t)p) & 15) == 0;
}

struct SpecPlan {
    SpecGrid G;
    int fields = kFftMaxFields;   // that the hybrid correction has room for
    size_t bytes = 0;             // the query's size, with room for all three
    size_t least = 0;
};

// validates the shape and carves the workspace (ws == nullptr: sizes only)
int spec_plan(const int* n, int isolated, void* ws, size_t ws_bytes, SpecPlan& S) {
    int rc = spec_grid_init(n, isolated, S.G);
    if (rc) return rc;
    size_t off = 0;
    spec_grid_carve(S.G, (char*)ws, off);
    off = align256(off);
    S.G.W = ws ? (double2*)((char*)ws + off) : nullptr;
    const SpecGrid& G = S.G;
    // the size that callers may keep is that of one n0 x n1 x P2 and two n0 x P1 x P2 complex arrays.  The hybrid
    // correction's components take three fields; with rows of two modes (one cell along z, isolated) these can
    // be more, and in the smaller size it forms the components one after the other, from the spectrum kept in
    // the first field into a second (100 x 100 x 1: 44 us in three fields, 80 us in two)
    const size_t w1 = sizeof(double2) * (size_t)G.n[0] * G.n[1] * G.P[2];
    const size_t w2 = sizeof(double2) * (size_t)G.n[0] * G.P[1] * G.P[2];
    const size_t full = align256(w1) + align256(w2) + w2, field = sizeof(double2) * G.field();
    S.least = align256(off + std::max(2 * field, full));
    S.bytes = std::max(S.least, align256(off + kFftMaxFields * field));
    S.fields = ws_bytes >= S.bytes ? kFftMaxFields : 2;
    return MG_OK;
}

int check_ws(const SpecPlan& S, void* ws, size_t ws_bytes) {
    if (!ws || ws_bytes < S.least)
        return report_error(MG_EINVAL, ("workspace too small: need " + std::to_string(S.bytes)).c_str());
    if (((uintptr_t)ws) & 255) return report_error(MG_EINVAL, "workspace must be 256-byte aligned");
    return MG_OK;
}

}  // namespace

int spec_grid_init(const int* n, int isolated, SpecGrid& S) {
    if (!n) return report_error(MG_EINVAL, "shape is NULL");
    for (int a = 0; a < 3; ++a) {
        if (n[a] < 1) return report_error(MG_EINVAL, "every axis needs at least one cell");
        const int P = isolated ? pad_len(n[a]) : n[a];
        const int lg = log2_exact(P);
        if (lg < 1 || lg > kFftMaxLgN)
            return report_error(MG_EINVAL, isolated ? "isolated transforms need n <= 512 on every axis"
                                                    : "periodic transforms need power-of-two n in 2..1024");
        S.n[a] = n[a];
        S.P[a] = P;
        S.lg[a] = lg;
    }
    S.lgtw = std::max(S.lg[0], std::max(S.lg[1], S.lg[2]));
    // rows start on 128-byte lines, and their length is no power of two
    const int M = S.P[2] / 2;
    S.zs = M < 16 ? M + 1 : M + 8;
    return MG_OK;
}

void spec_grid_carve(SpecGrid& S, char* base, size_t& off) {
    auto take = [&](size_t bytes) -> void* {
        off = align256(off);
        void* p = base ? (void*)(base + off) : nullptr;
        off += bytes;
        return p;
    };
    S.tw = (double2*)take(sizeof(double2) << S.lgtw);
    for (int a = 0; a < 3; ++a) S.tab[a] = (double*)take(4 * sizeof(double) * (size_t)S.P[a]);
}

hipError_t spec_grid_prepare(const SpecGrid& S, int kind, int lap_order, int grad_order, hipStream_t st) {
    return launch_spec_tables(S.tw, S.lgtw, S.tab[0], S.tab[1], S.tab[2], S.P, kind, lap_order, grad_order, st);
}

// z then y forward passes of a real field into W (prep: formed from the field while it is read)
hipError_t spec_forward_zy(const SpecGrid& S, const double* in, const SpecField& f, const ConvPrep* prep,
                           hipStream_t st) {
    FftPass z = pass_z(S, f, 1);
    z.in_lo = f.lo[2];
    z.in_hi = f.hi[2];
    z.rin[0] = in;
    z.vec = by_pairs(f, in) ? 1 : 0;
    ConvPrep C;
    if (prep) {
        C = *prep;
        C.x0 = f.lo[0];
        C.y0 = f.lo[1];
    }
    const hipError_t e = launch_fft_z_forward(z, prep ? &C : nullptr, st);
    if (e != hipSuccess) return e;
    FftPass y = pass_y(S, f, 1);
    y.in_lo = f.lo[1];
    y.in_hi = f.hi[1];
    y.out_hi = S.P[1];
    return launch_fft_lines(y, kFftForward, 0, st);
}

// forward x pass: the spectrum (every point) into out, complex (op kFftForward) or its real part
// (kFftRe), layout [P0][P1][zs]
hipError_t spec_x_spectrum(const SpecGrid& S, int op, void* out, hipStream_t st) {
    FftPass x = pass_x(S);
    x.in_hi = S.n[0];
    x.out_hi = S.P[0];
    x.out = out;
    return launch_fft_lines(x, op, 0, st);
}

// x pass in place: forward from the field's planes `in`, multiply, inverse to the planes of `out`
// (op kFftFwdSymInv; kFftHybrid: into the three components of the correction, W and the two fields
// after it; kFftHybridOne: component m.comp, into the field after W)
hipError_t spec_x_pass(const SpecGrid& S, int op, const SpecMul& m, const SpecField& in, const SpecField& out,
                       hipStream_t st) {
    FftPass x = pass_x(S);
    x.comp = m.comp;
    if (op == kFftHybridOne) x.out = S.W + S.field();
    x.in_lo = in.lo[0];
    x.in_hi = in.hi[0];
    x.out_lo = out.lo[0];
    x.out_hi = out.hi[0];
    x.tab = m.tab;
    x.tab_si = (long long)S.P[1] * S.zs;
    x.tab_sa = S.zs;
    if (m.coarse) {
        x.csp = m.csp;
        x.csp_zs = m.coarse->zs;
        for (int a = 0; a < 3; ++a) x.cn[a] = m.coarse->P[a];
    }
    // the inverse transform's 1 / (P0 P1 P2) rides on the multiplier
    x.sym_scale = m.scale / ((double)S.P[0] * (double)S.P[1] * (double)S.P[2]);
    x.fine_scale = m.fine_scale / ((double)S.P[0] * (double)S.P[1] * (double)S.P[2]);
    return launch_fft_lines(x, op, m.sym, st);
}

// y then z inverse passes of the nf fields in W -> real outputs, stored or added
hipError_t spec_inverse_yz(const SpecGrid& S, double* const* out, int nf, const SpecField& f, bool add,
                           hipStream_t st) {
    // Fields that fit the 256 MB Infinity Cache together share their launches; larger ones go one
    // after the other, so that the z pass finds in the cache what the y pass has just written.
    if (nf > 1 && sizeof(double2) * S.field() * nf > ((size_t)192 << 20)) {
        SpecGrid one = S;
        for (int k = 0; k < nf; ++k, one.W += S.field()) {
            const hipError_t e = spec_inverse_yz(one, out + k, 1, f, add, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    FftPass y = pass_y(S, f, nf);
    y.in_hi = S.P[1];
    y.out_lo = f.lo[1];
    y.out_hi = f.hi[1];
    const hipError_t e = launch_fft_lines(y, kFftInverse, 0, st);
    if (e != hipSuccess) return e;
    FftPass z = pass_z(S, f, nf);
    z.out_lo = f.lo[2];
    z.out_hi = f.hi[2];
    for (int k = 0; k < nf; ++k) {
        z.rout[k] = out[k];
        z.vec |= by_pairs(f, out[k]) ? 1 << k : 0;
    }
    return launch_fft_z_inverse(z, add, st);
}

}  // namespace mgic

using namespace mgic;

extern "C" {

size_t spec_workspace_bytes(const int n[3], int isolated) {
    SpecPlan S;
    if (spec_plan(n, isolated, nullptr, 0, S)) return 0;
    return S.bytes;
}

int spec_deconvolve(const int n[3], int kind, int isolated, const double* f, double* out, void* ws, size_t ws_bytes,
                    void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (kind != SPEC_FV_DECONV && kind != SPEC_SG_DECONV) return report_error(MG_EINVAL, "unknown deconvolution kind");
    if (!f || !out) return report_error(MG_EINVAL, "f or out is NULL");
    SpecPlan S;
    int rc = spec_plan(n, isolated, nullptr, 0, S);
    if (rc) return rc;
    if ((rc = check_ws(S, ws, ws_bytes))) return rc;
    spec_plan(n, isolated, ws, ws_bytes, S);
    const SpecGrid& G = S.G;
    SP_HIP(spec_grid_prepare(G, kind == SPEC_FV_DECONV ? kSpecFv : kSpecSg, 2, 4, st));
    SpecMul m;
    m.sym = kSymSeparable;
    const SpecField F(G.n);
    SP_HIP(spec_forward_zy(G, f, F, nullptr, st));
    SP_HIP(spec_x_pass(G, kFftFwdSymInv, m, F, F, st));
    SP_HIP(spec_inverse_yz(G, &out, 1, F, false, st));
    return MG_OK;
}

int spec_poisson(const int n[3], double h, int order, const double* f, double* u, void* ws, size_t ws_bytes,
                 void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (order != 2 && order != 4 && order != 6) return report_error(MG_EINVAL, "order must be 2, 4 or 6");
    if (!(h > 0) || !std::isfinite(h)) return report_error(MG_EINVAL, "h must be positive and finite");
    if (!f || !u) return report_error(MG_EINVAL, "f or u is NULL");
    SpecPlan S;
    int rc = spec_plan(n, 0, nullptr, 0, S);
    if (rc) return rc;
    if ((rc = check_ws(S, ws, ws_bytes))) return rc;
    spec_plan(n, 0, ws, ws_bytes, S);
    const SpecGrid& G = S.G;
    SP_HIP(spec_grid_prepare(G, kSpecPoisson, order, 4, st));
    SpecMul m;
    m.sym = kSymInvLap;
    m.scale = h * h;
    const SpecField F(G.n);
    SP_HIP(spec_forward_zy(G, f, F, nullptr, st));
    SP_HIP(spec_x_pass(G, kFftFwdSymInv, m, F, F, st));
    SP_HIP(spec_inverse_yz(G, &u, 1, F, false, st));
    return MG_OK;
}

int lpt_hybrid_correction(const int n[3], double h, int isolated, int lap_order, int grad_order, double scale,
                          const double* f, double* const* out3, void* ws, size_t ws_bytes, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    if (lap_order != 2 && lap_order != 4 && lap_order != 6)
        return report_error(MG_EINVAL, "lap_order must be 2, 4 or 6");
    if (grad_order != 4 && grad_order != 6) return report_error(MG_EINVAL, "grad_order must be 4 or 6");
    if (!(h > 0) || !std::isfinite(h)) return report_error(MG_EINVAL, "h must be positive and finite");
    if (!std::isfinite(scale)) return report_error(MG_EINVAL, "scale must be finite");
    if (!f || !out3 || !out3[0] || !out3[1] || !out3[2]) return report_error(MG_EINVAL, "f or an output is NULL");
    SpecPlan S;
    int rc = spec_plan(n, isolated, nullptr, 0, S);
    if (rc) return rc;
    if ((rc = check_ws(S, ws, ws_bytes))) return rc;
    spec_plan(n, isolated, ws, ws_bytes, S);
    const SpecGrid& G = S.G;
    SP_HIP(spec_grid_prepare(G, kSpecHybrid, lap_order, grad_order, st));
    SpecMul m;
    m.scale = scale * h;
    const SpecField F(G.n);
    SP_HIP(spec_forward_zy(G, f, F, nullptr, st));
    if (S.fields == kFftMaxFields) {
        SP_HIP(spec_x_pass(G, kFftHybrid, m, F, F, st));
        SP_HIP(spec_inverse_yz(G, out3, 3, F, true, st));
        return MG_OK;
    }
    SpecGrid second = G;
    second.W += G.field();
    for (int c = 0; c < 3; ++c) {
        m.comp = c;
        SP_HIP(spec_x_pass(G, kFftHybridOne, m, F, F, st));
        SP_HIP(spec_inverse_yz(second, out3 + c, 1, F, true, st));
    }
    return MG_OK;
}

}  // extern "C"
