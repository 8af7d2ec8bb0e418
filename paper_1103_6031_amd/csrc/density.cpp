// Host side of the multi-scale density (Hahn & Abel 2011, Sections 2.1-2.3 and 3.5.3): kernels
// per level, mode-preserving noise refinement and the nested convolutions, scheduled on the
// three-pass FFT of k_fft.hip and the grid kernels of k_density.hip.
//
// Levels: 0 is the periodic base (N^3); patch p has n_p cells per axis and the padded domain D'_p
// of 2 n_p cells per axis centred on it (the patch at [n_p/2, 3 n_p/2) of D'_p).  Per level the
// workspace holds the noise (N^3, or (2 n_p)^3 on D'_p) and the kernel grid, which is transformed
// in place into its (real) spectrum.  Convolutions are circular on the base or on D'_p.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "spec_internal.h"
#include "mgic.h"

namespace mgic {

namespace {

#define DN_HIP(call)                                                                             \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess) {                                                                  \
            (void)hipGetLastError();                                                             \
            return report_error(MG_EHIP, (std::string(#call) + ": " + hipGetErrorString(e_)).c_str()); \
        }                                                                                        \
    } while (0)

size_t cells3(const int* n) { return (size_t)n[0] * n[1] * n[2]; }

struct DensLevel {
    int n[3];        // own cells
    int off[3];      // in parent cells (patches)
    int D[3];        // noise / kernel grid: N (base) or 2 n (patch)
    double h;
    double* mu = nullptr;    // noise, D cells
    double* T = nullptr;     // kernel grid, then its spectrum, D cells
    SpecGrid G;              // transforms on D (periodic)
    SpecGrid R;              // the parent region under D' (n cells per axis, periodic) - patches
};

struct DensPlan {
    int nl = 0;
    std::vector<DensLevel> L;
    double* reg = nullptr;       // gathered parent region (max n^3)
    double2* csp = nullptr;      // its spectrum (half of the modes)
    double* b = nullptr;         // a convolution's output on D' (max (2n)^3)
    double* carry0 = nullptr;    // the base's coarse contribution (N^3)
    double* carryA = nullptr;    // coarse contributions on patches (max n^3), ping-pong
    double* carryB = nullptr;
    size_t bytes = 0;
};

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

int dens_plan(const mg_hier* H, void* ws, DensPlan& P) {
    if (!H) return report_error(MG_EINVAL, "hierarchy is NULL");
    if (H->nlev < 1 || H->nlev > MG_MAX_LEVELS) return report_error(MG_EINVAL, "nlev out of range");
    const mg_level& b = H->lev[0];
    const int N = b.n[0];
    if (b.n[1] != N || b.n[2] != N) return report_error(MG_EINVAL, "base must be cubic");
    if (log2_exact(N) < 1 || N > 1024) return report_error(MG_EINVAL, "base must be a power of two in 2..1024");
    if (!(b.h > 0) || !std::isfinite(b.h)) return report_error(MG_EINVAL, "base spacing must be positive");
    P.nl = H->nlev;
    P.L.assign(P.nl, DensLevel());
    for (int l = 0; l < P.nl; ++l) {
        const mg_level& v = H->lev[l];
        DensLevel& D = P.L[l];
        D.h = v.h;
        for (int a = 0; a < 3; ++a) {
            D.n[a] = v.n[a];
            D.off[a] = l ? v.off[a] : 0;
            D.D[a] = l ? 2 * v.n[a] : N;
        }
        if (l == 0) continue;
        const DensLevel& Q = P.L[l - 1];
        if (std::fabs(v.h - 0.5 * Q.h) > 1e-12 * Q.h) return report_error(MG_EINVAL, "patch spacing must be half its parent's");
        for (int a = 0; a < 3; ++a) {
            const int n = v.n[a], o = v.off[a];
            if (n < 4 || log2_exact(n) < 0 || 2 * n > 1024)
                return report_error(MG_EINVAL, "patch sizes must be powers of two in 4..512");
            if (l == 1) {
                if (o < 0 || o + n / 2 > N || n / 2 > N - 2 || n > N)
                    return report_error(MG_EINVAL, "first patch not properly nested in the base");
            } else {
                if (o < 4 || o + n / 2 > Q.n[a] - 4) return report_error(MG_EINVAL, "patch not properly nested in its parent");
                if (o - n / 4 < 0 || o + 3 * n / 4 > Q.n[a])
                    return report_error(MG_EINVAL, "padded domain of a patch leaves its parent");
            }
        }
    }
    size_t off = 0;
    char* base = (char*)ws;
    auto take = [&](size_t bytes) -> void* {
        off = al256(off);
        void* p = base ? (void*)(base + off) : nullptr;
        off += bytes;
        return p;
    };
    size_t w = 0, maxn = 0, maxd = 0, maxs = 0;
    for (int l = 0; l < P.nl; ++l) {
        DensLevel& D = P.L[l];
        int rc = spec_grid_init(D.D, 0, D.G);
        if (rc) return rc;
        spec_grid_carve(D.G, base, off);
        w = std::max(w, D.G.field());
        D.mu = (double*)take(sizeof(double) * cells3(D.D));
        D.T = (double*)take(sizeof(double) * cells3(D.D));
        if (l) {
            rc = spec_grid_init(D.n, 0, D.R);
            if (rc) return rc;
            spec_grid_carve(D.R, base, off);
            w = std::max(w, D.R.field());
            maxs = std::max(maxs, D.R.field());
            maxn = std::max(maxn, cells3(D.n));
            maxd = std::max(maxd, cells3(D.D));
        }
    }
    double2* W = (double2*)take(sizeof(double2) * w);
    for (DensLevel& D : P.L) D.G.W = D.R.W = W;
    const size_t nb = cells3(P.L[0].D);
    P.carry0 = (double*)take(sizeof(double) * nb);
    if (P.nl > 1) {
        P.reg = (double*)take(sizeof(double) * maxn);
        P.csp = (double2*)take(sizeof(double2) * maxs);
        P.b = (double*)take(sizeof(double) * maxd);
        P.carryA = (double*)take(sizeof(double) * maxn);
        P.carryB = (double*)take(sizeof(double) * maxn);
    }
    P.bytes = al256(off);
    return MG_OK;
}

// the parent's noise (or any parent array of the same layout) as seen from patch l: the box of
// parent cells starting at lo (in the parent's own cells)
DensBox parent_box(const DensPlan& P, int l, const int* lo) {
    DensBox B;
    const DensLevel& Q = P.L[l - 1];
    for (int a = 0; a < 3; ++a) {
        B.pd[a] = Q.D[a];
        B.po[a] = l == 1 ? 0 : Q.n[a] / 2;
        B.lo[a] = lo[a];
    }
    B.wrap = l == 1 ? Q.n[0] : 0;
    return B;
}

// a parent array of the parent's own cells (no padding: the base, or a patch's n^3 array)
DensBox parent_plain_box(const DensPlan& P, int l, const int* lo) {
    DensBox B;
    const DensLevel& Q = P.L[l - 1];
    for (int a = 0; a < 3; ++a) {
        B.pd[a] = Q.n[a];
        B.po[a] = 0;
        B.lo[a] = lo[a];
    }
    B.wrap = l == 1 ? Q.n[0] : 0;
    return B;
}

int run_density(const DensPlan& P, const double* table, double dr, int subgrid, const double* const* xi,
                double* const* delta, hipStream_t st) {
    const int top = P.nl - 1;
    // ---- kernels, finest first; each grid becomes its spectrum once the next coarser is built
    DN_HIP(launch_kernel_direct(P.L[top].T, P.L[top].D, P.L[top].h, table, dr, subgrid, st));
    for (int l = top; l >= 0; --l) {
        const DensLevel& D = P.L[l];
        if (l > 0) {
            const DensLevel& Q = P.L[l - 1];
            DN_HIP(launch_kernel_restrict(Q.T, Q.D, Q.h, D.T, D.D, table, dr, st));
        }
        DN_HIP(spec_grid_prepare(D.G, l > 0 ? kSpecReplace : 0, 2, 4, st));
        DN_HIP(spec_forward_zy(D.G, D.T, SpecField(D.D), nullptr, st));
        DN_HIP(spec_x_spectrum(D.G, kFftRe, D.T, st));
    }
    // ---- noise: scale, refine top-down (mode replacement), then reverse Hoffman-Ribak bottom-up
    DN_HIP(launch_divide(P.L[0].mu, xi[0], cells3(P.L[0].D), std::pow(P.L[0].h, 1.5), st));
    for (int l = 1; l <= top; ++l) {
        const DensLevel& D = P.L[l];
        int lo[3];
        for (int a = 0; a < 3; ++a) lo[a] = D.off[a] - D.n[a] / 4;
        DN_HIP(launch_gather(P.reg, D.n, P.L[l - 1].mu, parent_box(P, l, lo), st));
        DN_HIP(spec_grid_prepare(D.R, 0, 2, 4, st));
        DN_HIP(spec_forward_zy(D.R, P.reg, SpecField(D.n), nullptr, st));
        DN_HIP(spec_x_spectrum(D.R, kFftForward, P.csp, st));
        const SpecField F(D.D);
        SpecMul m;   // the noise's own scale rides on the modes that it keeps
        m.sym = kSymReplace;
        m.csp = P.csp;
        m.coarse = &D.R;
        m.fine_scale = 1.0 / std::pow(D.h, 1.5);
        DN_HIP(spec_forward_zy(D.G, xi[l], F, nullptr, st));
        DN_HIP(spec_x_pass(D.G, kFftFwdSymInv, m, F, F, st));
        DN_HIP(spec_inverse_yz(D.G, &D.mu, 1, F, false, st));
    }
    for (int l = top; l >= 1; --l) {
        const DensLevel& D = P.L[l];
        const int m[3] = {D.n[0] / 2, D.n[1] / 2, D.n[2] / 2};
        const int co[3] = {D.n[0] / 2, D.n[1] / 2, D.n[2] / 2};
        DN_HIP(launch_restrict_mean(P.L[l - 1].mu, parent_box(P, l, D.off), m, D.mu, D.D, co, st));
    }
    // ---- convolutions
    auto convolve = [&](const DensLevel& D, const SpecField& in, const double* mu, const ConvPrep* prep,
                        const SpecField& to, double* out, bool add) -> hipError_t {
        SpecMul m;
        m.sym = kSymTable;
        m.scale = D.h * D.h * D.h;
        m.tab = D.T;
        hipError_t e = spec_forward_zy(D.G, mu, in, prep, st);
        if (e == hipSuccess) e = spec_x_pass(D.G, kFftFwdSymInv, m, in, to, st);
        if (e == hipSuccess) e = spec_inverse_yz(D.G, &out, 1, to, add, st);
        return e;
    };
    {
        const DensLevel& B = P.L[0];
        const SpecField F(B.D);
        DN_HIP(convolve(B, F, B.mu, nullptr, F, delta[0], false));
        if (top >= 1) {   // the noise outside the first patch, for what the patches receive
            ConvPrep open;
            open.mode = kPrepOpen;
            for (int a = 0; a < 3; ++a) {
                open.lo[a] = P.L[1].off[a];
                open.hi[a] = P.L[1].off[a] + P.L[1].n[a] / 2;
            }
            DN_HIP(convolve(B, F, B.mu, &open, F, P.carry0, false));
        }
    }
    const double* src = P.carry0;
    double* dst = P.carryA;
    for (int l = 1; l <= top; ++l) {
        const DensLevel& D = P.L[l];
        int lo[3], half[3];
        for (int a = 0; a < 3; ++a) {
            lo[a] = D.off[a] - D.n[a] / 4;
            half[a] = D.n[a] / 2;
        }
        const bool next = l < top;
        const SpecField F(D.D), own(D.n, half, D.n);   // D', and the patch's cells in it
        // coarse contributions carried down; the noise inside the patch and minus its parent's on the
        // padding adds this level's density to them
        DN_HIP(launch_interp_cons(delta[l], next ? dst : nullptr, D.n, src, parent_plain_box(P, l, D.off), st));
        ConvPrep prep;
        prep.mode = kPrepSelf;
        prep.par = P.L[l - 1].mu;
        prep.pb = parent_box(P, l, lo);
        for (int a = 0; a < 3; ++a) {
            prep.lo[a] = half[a];
            prep.hi[a] = half[a] + D.n[a];
        }
        DN_HIP(convolve(D, F, D.mu, &prep, own, delta[l], true));
        // delta_bnd restricted onto the parent cells under D' that the patch does not cover
        prep.mode = kPrepBnd;
        DN_HIP(convolve(D, F, D.mu, &prep, F, P.b, false));
        DN_HIP(launch_restrict_add(delta[l - 1], parent_plain_box(P, l, lo), P.b, D.n, st));
        if (next) {   // the noise inside the patch and outside the next one, for what that receives
            ConvPrep open;
            open.mode = kPrepOpen;
            for (int a = 0; a < 3; ++a) {
                open.lo[a] = half[a] + P.L[l + 1].off[a];
                open.hi[a] = open.lo[a] + P.L[l + 1].n[a] / 2;
            }
            const double* mu = D.mu + ((size_t)half[0] * D.D[1] + half[1]) * D.D[2] + half[2];
            DN_HIP(convolve(D, SpecField(D.n, half, D.D), mu, &open, own, dst, true));
            src = dst;
            dst = dst == P.carryA ? P.carryB : P.carryA;
        }
    }
    // ---- composite: covered coarse cells := mean of their children, finest first
    for (int l = top; l >= 1; --l) {
        const DensLevel& D = P.L[l];
        const int m[3] = {D.n[0] / 2, D.n[1] / 2, D.n[2] / 2};
        const int co[3] = {0, 0, 0};
        DN_HIP(launch_restrict_mean(delta[l - 1], parent_plain_box(P, l, D.off), m, delta[l], D.n, co, st));
    }
    return MG_OK;
}

}  // namespace

}  // namespace mgic

using namespace mgic;

extern "C" {

size_t ic_density_workspace_bytes(const mg_hier* hier) {
    DensPlan P;
    if (dens_plan(hier, nullptr, P)) return 0;
    return P.bytes;
}

int ic_multiscale_density(const mg_hier* hier, const double* radial, int nradial, double dr, int subgrid,
                          const double* const* xi, double* const* delta, void* ws, size_t ws_bytes, void* stream) {
    hipStream_t st = (hipStream_t)stream;
    DensPlan P;
    int rc = dens_plan(hier, nullptr, P);
    if (rc) return rc;
    if (!radial || nradial < 2) return report_error(MG_EINVAL, "the radial table needs at least 2 entries");
    if (!(dr > 0) || !std::isfinite(dr)) return report_error(MG_EINVAL, "dr must be positive and finite");
    if (!xi || !delta) return report_error(MG_EINVAL, "noise or output pointer array is NULL");
    for (int l = 0; l < P.nl; ++l)
        if (!xi[l] || !delta[l]) return report_error(MG_EINVAL, "a level pointer is NULL");
    // the largest radius any kernel grid samples: the base at |D| <= sqrt(3) N/2 H, a patch's
    // padded grid at sqrt(3) n h, plus the sub-cell offsets of the finest level
    double rmax = std::sqrt(3.0) * 0.5 * P.L[0].n[0] * P.L[0].h;
    for (int l = 1; l < P.nl; ++l) {
        const DensLevel& D = P.L[l];
        const double m = (double)std::max(D.n[0], std::max(D.n[1], D.n[2]));
        rmax = std::max(rmax, std::sqrt(3.0) * m * D.h);
    }
    rmax += std::sqrt(3.0) * 0.25 * P.L[P.nl - 1].h;
    if (rmax / dr >= (double)(nradial - 2))
        return report_error(MG_EINVAL, ("the radial table must reach r = " + std::to_string(rmax)).c_str());
    if (!ws || ws_bytes < P.bytes)
        return report_error(MG_EINVAL, ("workspace too small: need " + std::to_string(P.bytes)).c_str());
    if (((uintptr_t)ws) & 255) return report_error(MG_EINVAL, "workspace must be 256-byte aligned");
    dens_plan(hier, ws, P);
    return run_density(P, radial, dr, subgrid ? 1 : 0, xi, delta, st);
}

}  // extern "C"
