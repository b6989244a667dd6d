// internal.h -- data layout shared by the host runtime and the gfx950 kernels.
//
// Everything the kernels read lives in one caller-owned device buffer (the
// "geometry buffer"); GeomLayout holds the byte offset of each table.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace bemk {

constexpr int QMAX = 16;      // largest Gauss rule
constexpr int ROW_TILE = 256; // collocation rows per assembly workgroup
constexpr int COL_CHUNK = 32; // source elements per assembly workgroup
constexpr int NEAR_PART = 4;  // source elements per workgroup of the near-element launch
// |k r| below which the device Hankel evaluator uses the series (FP64 and FP32
// amplitude paths; the same values as in hankel_tables.h).  For Im k > 0.07 Re k (4
// degrees) the FP64 path keeps them to 7: between 6 and 7 the amplitude fits,
// made on the real axis, are good to 3e-14 at 4 degrees and 2e-12 at 10, the
// series to 2e-15; below 4 degrees the entries' error is that of the rest.
constexpr double XS_SERIES_F64 = 6.0, XS_SERIES_F32 = 4.0, XS_SERIES_WIDE = 7.0, WIDE_TAN = 0.07;
__host__ __device__ constexpr double series_radius(double kr, double ki)
{
    return ki > WIDE_TAN * kr ? XS_SERIES_WIDE : XS_SERIES_F64;
}
constexpr int MAX_DIRS = 4096;

// Largest Im k / Re k of a lossy medium: tan(10 degrees).
constexpr double MAX_TAN_ARG_K = 0.17632698070846498;

// One boundary element (128 bytes).  Normal = left normal of the travel
// direction a -> b.
struct ElemRec {
    double cx, cy;     // midpoint = collocation point
    double tx, ty;     // unit tangent (b - a) / h
    double nx, ny;     // unit normal (-ty, tx)
    double close2[2];  // ExpHead::close2 in the domains dom_left and dom_right; without expansion (5/2 h)^2
    double h;          // length |b - a|
    double ax, ay;     // first node
    double bx, by;     // second node
    double pad[3];
};

// Expansion record of one element in the domain on one side of it (the sums of
// its Gauss rule from one Hankel evaluation at its midpoint, assemble.hip):
// EXP_HEAD doubles of squared distance limits (infinite where the element is
// too long against the wavelength, except for the last two), then the
// coefficients by order: order 0 has (S, Tt), an odd order (Gt, Gn), an even one
// (S, Tt, Tn).
constexpr int EXP_HEAD = 12, EXP_LMAX = 20, EXP_NCOEF = 52, EXP_NTERMS = 14;
__host__ __device__ constexpr int exp_pos(int m)
{
    return m == 0 ? 0 : (m & 1) ? 2 + 5 * (m / 2) : 4 + 5 * (m / 2 - 1);
}
static_assert(exp_pos(EXP_LMAX) + 3 == EXP_NCOEF, "coefficients of the orders 0 .. EXP_LMAX");
struct ExpHead {
    double close2;                     // below it: no expansion (order 20 leaves too much)
    double near64;                     // below it: near launch of the FP64 assembly (close2, series radius)
    double lim8, lim10, lim12, lim16;  // beyond it: order 8, 10, 12, 16 suffices
    double near32;                     // the same for the FP32 assembly (remainder 1e-9)
    double lim32_4, lim32_6, lim32_8;
    double take64, take32;             // below it: near launch; as near64, near32, but for an element
                                       // without expansion (XS/|k| + h/2)^2
};
constexpr int EXP_H_CLOSE = 0, EXP_H_NEAR64 = 1, EXP_H_LIM = 2, EXP_H_NEAR32 = 6, EXP_H_LIM32 = 7,
              EXP_H_TAKE64 = 10, EXP_H_TAKE32 = 11;
static_assert(sizeof(ExpHead) == EXP_HEAD * sizeof(double), "head of an expansion record");
// With x = (h/2)/r the remainder of order L is about x^L, and about
// (kh/4)^L / (L+1)! where kr is large: the largest x and |k| h/2 at which the
// remainder of every sum, relative to its leading term, stays below 4e-17
// (FP32: 1e-9) for real k (gen_expansion_limits.py).  At arg k = 10 degrees the
// vector sums leave up to 1.4e-16, the end-point differences 2.3e-16 (1e-9 and
// 1.7e-9).
constexpr double EXP_X8 = 0.0087, EXP_X10 = 0.0223, EXP_X12 = 0.0415, EXP_X16 = 0.0855, EXP_X20 = 0.128;
constexpr double EXP_KA8 = 0.074, EXP_KA10 = 0.228, EXP_KA12 = 0.495, EXP_KA16 = 1.36, EXP_KA_MAX = 2.55;
constexpr double EXP32_X4 = 0.0054, EXP32_X6 = 0.0306, EXP32_X8 = 0.0725, EXP32_X16 = 0.2;
constexpr double EXP32_KA4 = 0.026, EXP32_KA6 = 0.206, EXP32_KA8 = 0.615;
// Shorter elements take the Gauss rule: H_20 at their close distance (7e264 at
// this limit) and the coefficients (1e-299) would leave the range of a double.
constexpr double EXP_KA_MIN = 1e-13;

// Inputs of a domain as given by the caller (complex numbers as re, im).
struct DomIn {
    double k[2];
    double bm[2];
    int has_bm;
    int pad;
};

struct GlobalIn {
    double alpha[2];
    double beta[2];
    int has_alpha, has_beta, form, n_dom;
};

// Derived per-domain constants (computed on the device).
struct DomConst {
    double k[2];     // wavenumber
    double eps[2];   // (k / k0)^2
    double c[2];     // Burton-Miller coefficient alpha / eps (or the caller's)
    double beta[2];  // scaling of the standard-type rows
    int cplx;        // Im k != 0
    int pad;
};

// Per-wavenumber constants of the device Hankel evaluator (hankel_dev.h): the
// polynomial coefficients are compile-time constants, the wavenumber enters
// through the arguments w = (XS/k)^2 / r^2 and t = (k/2)^2 r^2.
struct WaveConst {
    double kr, ki;
    double r2_small;            // (XS / |k|)^2: below it the ascending series
    double wr, wi;              // (XS / k)^2
    double ur, ui;              // XS / k
    double tr, ti;              // (k / 2)^2
    double hr, hi;              // k / 2
    double lkr, lki;            // ln(k / 2)
    double y1r, y1i;            // -2 / (pi k)
    double ampr, ampi;          // sqrt(2 / (pi k))
    double tkr, tki;            // 2 / k
};

// Interface plan (host-computed integer bookkeeping).
struct IfacePlan {
    int off, count;   // element range
    int dl, dr;       // domain the normal enters / leaves
    int bm_r;         // the dom_right equation is of Burton-Miller type
    int row_l, row_r; // first row of the dom_left / dom_right equation block
    int pad;
};

// A tile of consecutive elements of one interface.
struct Tile {
    int iface, start, count, pad;
};

struct GeomLayout {
    size_t nodes, elnodes, elem, expn, gl, dom_in, glob_in, dom, wave, self,
        iface, rtiles, cchunks, sigma, elif, vtiles, npairs, total;
    int exp_stride, exp_cplx;  // doubles per expansion record; 1 if some wavenumber is complex
};

}  // namespace bemk
