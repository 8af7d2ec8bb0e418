// Internal declarations of the spectral side of the library: the three-pass FFT (k_fft.hip), its
// host pipelines (spectral.cpp) and the multi-scale density (k_density.hip, density.cpp).
// Not part of the public ABI (see include/mgic.h).
#pragma once

#include "mg_internal.h"

namespace mgic {

// ---- three-dimensional FFTs of real fields (k_fft.hip) ------------------------------------------
constexpr int kFftMaxLgN = 10;                       // transforms of length 2 .. 1024
constexpr int kFftMaxFields = 3;                     // fields transformed together
enum { kFftForward = 0, kFftInverse = 1, kFftFwdSymInv = 2, kFftRe = 3, kFftHybrid = 4, kFftHybridOne = 5 };
enum { kSymSeparable = 1, kSymTable = 2, kSymReplace = 5, kSymInvLap = 6 };
enum { kSpecFv = 1, kSpecSg = 2, kSpecHybrid = 3, kSpecReplace = 4, kSpecPoisson = 5 };
// one pass of batched 1-D transforms over nf fields fs complex points apart in the spectrum buffer.
// Strided passes: line (a, b), a < na, b <= 2^lgM, holds point i at a*sa + b + i*si; its points
// in_lo <= i < in_hi are read (the rest is zero), of the output out_lo <= i < out_hi are stored.
// z passes: na lines, `rows` of each x plane (planes `plane` rows of zs points apart in the buffer,
// rsx apart in the real array, real lines rsy apart); the array holds points in_lo .. in_hi
// (inverse: out_lo .. out_hi) of a line.
struct FftPass {
    int lgN = 0, lgM = 0, lgtw = 0;
    int in_lo = 0, in_hi = 0, out_lo = 0, out_hi = 0;
    int na = 0, nf = 1, rows = 1, zs = 0, plane = 0;
    long long in_sa = 0, in_si = 1, out_sa = 0, out_si = 1, fs = 0, rsx = 0, rsy = 0;
    const void* in = nullptr;
    void* out = nullptr;
    const double* rin[kFftMaxFields] = {nullptr, nullptr, nullptr};
    double* rout[kFftMaxFields] = {nullptr, nullptr, nullptr};
    int vec = 0;                    // bit f: field f's real lines can be accessed as 16-byte pairs
    const double2* tw = nullptr;
    // multiplier of the fused x pass: element (kx, ky, kz) = (point, a, b)
    const double* tab_x = nullptr;
    const double* tab_y = nullptr;
    const double* tab_z = nullptr;
    int sym_n[3] = {0, 0, 0};
    const double* tab = nullptr;
    long long tab_si = 0, tab_sa = 0;
    const double2* csp = nullptr;   // kSymReplace: the coarse region's spectrum, cn[0] x cn[1] x csp_zs
    int cn[3] = {0, 0, 0};
    int csp_zs = 0;
    int comp = 0;                   // kFftHybridOne: the component
    double sym_scale = 1.0;
    double fine_scale = 1.0;        // kSymReplace: the scale of the modes that are kept
};
// a box of cells of a parent array: array dims pd, the parent's own cells start at po inside the
// array, the box starts at lo in the parent's own cells; wrap > 0: periodic with wrap cells per axis
struct DensBox {
    int pd[3] = {0, 0, 0};
    int po[3] = {0, 0, 0};
    int lo[3] = {0, 0, 0};
    int wrap = 0;
};
// a convolution's input formed while it is read (k_fft.hip, conv_input): the cells lo <= . < hi of
// the transform grid are the patch (kPrepSelf, kPrepBnd) or the next patch's (kPrepOpen); the
// pass's first line is (x0, y0)
enum { kPrepSelf = 1, kPrepBnd = 2, kPrepOpen = 3 };
struct ConvPrep {
    int mode = 0;
    int x0 = 0, y0 = 0;
    int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    const double* par = nullptr;
    DensBox pb;
};
hipError_t launch_spec_tables(double2* tw, int lg, double* t0, double* t1, double* t2, const int P[3], int kind,
                              int lap_order, int grad_order, hipStream_t st);
hipError_t launch_fft_z_forward(const FftPass& A, const ConvPrep* prep, hipStream_t st);
hipError_t launch_fft_z_inverse(const FftPass& A, bool add, hipStream_t st);
hipError_t launch_fft_lines(const FftPass& A, int op, int sym, hipStream_t st);
// where a real field lies on a transform grid: its points lo <= . < hi, (x, y, z) at (x - lo0) sx +
// (y - lo1) sy + (z - lo2) of its array; lo2 is even
struct SpecField {
    int lo[3], hi[3];
    long long sx, sy;
    // n points per axis from `at` on (nullptr: the origin), in an array of `dims`
    SpecField(const int* n, const int* at, const int* dims) : sx((long long)dims[1] * dims[2]), sy(dims[2]) {
        for (int a = 0; a < 3; ++a) {
            lo[a] = at ? at[a] : 0;
            hi[a] = lo[a] + n[a];
        }
    }
    explicit SpecField(const int* n) : SpecField(n, nullptr, n) {}
};
// a 3-D transform grid: a field of n cells per axis transformed on P points per axis (P = n
// periodic, the zero-padded isolated length otherwise), with its twiddles, multiplier tables and
// the spectrum buffer W of its fields, each [n0][P1][zs] complex (kz = 0 .. P2 / 2 of a row used)
struct SpecGrid {
    int n[3] = {0, 0, 0};
    int P[3] = {0, 0, 0};
    int lg[3] = {0, 0, 0};
    int lgtw = 0;
    int zs = 0;
    double2* tw = nullptr;
    double* tab[3] = {nullptr, nullptr, nullptr};
    double2* W = nullptr;
    size_t field() const { return (size_t)n[0] * P[1] * zs; }   // complex points of a field
};
int spec_grid_init(const int* n, int isolated, SpecGrid& S);
void spec_grid_carve(SpecGrid& S, char* base, size_t& off);           // twiddles and tables
hipError_t spec_grid_prepare(const SpecGrid& S, int kind, int lap_order, int grad_order, hipStream_t st);
hipError_t spec_forward_zy(const SpecGrid& S, const double* in, const SpecField& f, const ConvPrep* prep,
                           hipStream_t st);
hipError_t spec_x_spectrum(const SpecGrid& S, int op, void* out, hipStream_t st);
// the multiplier of an x pass and what it needs
struct SpecMul {
    int sym = 0;
    double scale = 1.0;
    const double* tab = nullptr;           // kSymTable: [P0][P1][zs]
    const double2* csp = nullptr;          // kSymReplace: the coarse spectrum on the grid `coarse`
    const SpecGrid* coarse = nullptr;
    double fine_scale = 1.0;
    int comp = 0;                          // kFftHybridOne
};
hipError_t spec_x_pass(const SpecGrid& S, int op, const SpecMul& m, const SpecField& in, const SpecField& out,
                       hipStream_t st);
hipError_t spec_inverse_yz(const SpecGrid& S, double* const* out, int nf, const SpecField& f, bool add,
                           hipStream_t st);
// ---- multi-scale density (k_density.hip) -------------------------------------------------------
hipError_t launch_kernel_direct(double* T, const int* P, double h, const double* table, double dr, int subgrid,
                                hipStream_t st);
hipError_t launch_kernel_restrict(double* Tc, const int* P, double h, const double* Tf, const int* Pf,
                                  const double* table, double dr, hipStream_t st);
hipError_t launch_divide(double* out, const double* in, size_t n, double d, hipStream_t st);
hipError_t launch_gather(double* dst, const int* n, const double* src, const DensBox& b, hipStream_t st);
hipError_t launch_restrict_mean(double* parent, const DensBox& b, const int* m, const double* child, const int* cd,
                                const int* co, hipStream_t st);
hipError_t launch_interp_cons(double* out, double* out2, const int* n, const double* U, const DensBox& b,
                              hipStream_t st);
hipError_t launch_restrict_add(double* parent, const DensBox& b, const double* bnd, const int* n, hipStream_t st);
// error reporting shared by the host translation units (sets mg_last_error's message)
int report_error(int code, const char* msg);

}  // namespace mgic
