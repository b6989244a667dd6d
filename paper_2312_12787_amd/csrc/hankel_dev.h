// hankel_dev.h -- device evaluation of H0^(1)(k r) and H1^(1)(k r) for one
// wavenumber k (Im k >= 0) and many distances r > 0 (fundamental solution,
// eq. (fundamental_sol), and its derivative).
//
// Every polynomial has compile-time real coefficients (hankel_tables.h); the
// wavenumber enters only through the argument, so a launch keeps a handful
// of per-wavenumber constants (WaveConst) instead of coefficient tables.
//  * |k r| < XS: in t = (k r / 2)^2 = (k/2)^2 r^2 (DLMF 10.2.2, 10.8.1, 10.8.2)
//        J0 = J0(t),  Y0 = (2/pi)(ln(kr/2) + gamma) J0 + E0(t),
//        J1 = (kr/2) J1(t),  Y1 = -(2/pi)/(k r) + (2/pi) ln(kr/2) J1 + (kr/2) E1(t),
//    with ln(kr/2) = ln r + ln(k/2) (a real logarithm per lane) and the entire
//    functions J0, E0, J1, E1 from their ascending series for |k r| < 3, beyond
//    from their Taylor series about t = 5.5 (relative error of H0, real k, kr
//    from 0 to 6 in steps of 1, ascending series throughout / so: 0.8, 0.9, 2, 5,
//    15, 42 / 0.8, 0.9, 2, 2, 2, 2 1e-16);
//  * |k r| >= XS: H_nu = sqrt(2/(pi k)) r^{-1/2} e^{i(k r - nu pi/2 - pi/4)} P_nu,
//    P_nu = m_nu(w) + i (XS/(k r)) n_nu(w),  w = (XS/k)^2 / r^2, with m, n the
//    fitted amplitude polynomials.
// Real k: Horner in a real argument.  Complex k (lossy media): the same real
// polynomials at a complex argument z = x + i y by dividing out the quadratic
// z^2 - 2 x z + |z|^2 (Knuth's scheme): two multiply-adds per coefficient.
#pragma once

#include "fastmath_dev.h"
#include "hankel_tables.h"
#include "internal.h"

namespace bemk {

struct cd {
    double re, im;
};

__device__ __forceinline__ cd cmul(cd a, cd b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ cd cadd(cd a, cd b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ cd cscale(cd a, double s) { return {a.re * s, a.im * s}; }

// sum_m c[m] x^m, x real (c: an array of N coefficients, in any address space)
template <int N, class C, class T>
__device__ __forceinline__ T poly_n(const C& c, T x)
{
    T acc = c[N - 1];
#pragma unroll
    for (int m = N - 2; m >= 0; --m) acc = fma(acc, x, (T)c[m]);
    return acc;
}

// sum_m c[m] z^m at complex z = x + i y for real c: with R = 2x, S = |z|^2,
// b_{N-1} = c_{N-1}, b_{N-2} = c_{N-2} + R b_{N-1}, b_m = c_m + R b_{m+1} - S b_{m+2},
// p(z) = (x b_1 + c_0 - S b_2) + i y b_1.   (N >= 3)
template <int N, class C, class T>
__device__ __forceinline__ void poly_cplx_n(const C& c, T x, T y, T R, T S, T& pr, T& pi)
{
    T b2 = c[N - 1];
    T b1 = fma(R, b2, (T)c[N - 2]);
#pragma unroll
    for (int m = N - 3; m >= 1; --m) {
        const T b0 = fma(R, b1, fma(-S, b2, (T)c[m]));
        b2 = b1;
        b1 = b0;
    }
    pr = fma(x, b1, fma(-S, b2, (T)c[0]));
    pi = y * b1;
}

// The series coefficients as one object in device memory.  The general evaluator
// reads them through a pointer the compiler must reload on each call (scalar
// loads, nothing held in registers across a loop): its paths run rarely and
// would otherwise keep all of them resident.
template <int N>
struct SeriesTabs {
    double j0[N], e0[N], j1[N], e1[N];
};
struct HankelTabs {
    SeriesTabs<SERIES_NLOW> low;
    SeriesTabs<SERIES_NWIDE> mid;
};
constexpr HankelTabs make_hankel_tabs()
{
    HankelTabs t{};
    for (int m = 0; m < SERIES_NLOW; ++m) {
        t.low.j0[m] = LOW_J0[m];
        t.low.e0[m] = LOW_E0[m];
        t.low.j1[m] = LOW_J1[m];
        t.low.e1[m] = LOW_E1[m];
    }
    for (int m = 0; m < SERIES_NWIDE; ++m) {
        t.mid.j0[m] = MID_J0[m];
        t.mid.e0[m] = MID_E0[m];
        t.mid.j1[m] = MID_J1[m];
        t.mid.e1[m] = MID_E1[m];
    }
    return t;
}
static __device__ const HankelTabs g_hankel_tabs = make_hankel_tabs();
typedef const __attribute__((address_space(4))) HankelTabs* HankelTabsPtr;
__device__ __forceinline__ HankelTabsPtr hankel_tabs_fresh()
{
    HankelTabsPtr t = (HankelTabsPtr)&g_hankel_tabs;
    asm volatile("" : "+s"(t));  // opaque: loads through t are not hoisted out of loops
    return t;
}

// sum_m c[m] w^m from shared powers p[m] = w^m (p[0] unused), highest degree
// first.  The accumulator is the only register each step overwrites (Horner's
// rule overwrites a copy of the constant instead).  Used where 0 < w <= 1 and
// the |c[m]| of m >= 1 are small, so the order costs no accuracy.
template <int N, class C>
__device__ __forceinline__ double poly_pow(const C& c, const double* p)
{
    double acc = (double)c[N - 1] * p[N - 1];
#pragma unroll
    for (int m = N - 2; m >= 1; --m) acc = fma((double)c[m], p[m], acc);
    return acc + (double)c[0];
}

// The amplitude polynomials: LOW = false the FP64 fits (|k r| >= 6, 2e-16),
// LOW = true the short ones (|k r| >= 4, 7e-10) of the FP32 assembly; both
// evaluated in FP64.
template <bool LOW>
struct Amp;
template <>
struct Amp<false> {
    static constexpr int N = HANKEL_NC_F64;
    static constexpr double SCALE = 1.0;
    static constexpr const double (&m0)[N] = HANKEL_M0_F64, (&n0)[N] = HANKEL_N0_F64, (&m1)[N] = HANKEL_M1_F64,
                                  (&n1)[N] = HANKEL_N1_F64;
};
template <>
struct Amp<true> {
    static constexpr int N = HANKEL_NC_F32;
    static constexpr double SCALE = HANKEL_XS_F32 / HANKEL_XS_F64;
    static constexpr const float (&m0)[N] = HANKEL_M0_F32, (&n0)[N] = HANKEL_N0_F32, (&m1)[N] = HANKEL_M1_F32,
                                 (&n1)[N] = HANKEL_N1_F32;
};

// Large-argument form for |k r| >= XS, from r (+ rlo, the part of the distance
// that r lacks), 1/r and r^{-1/2}.  The phase phi = Re(k) r - pi/4 is reduced
// once for both orders:
//   H0 = A r^{-1/2} e^{i phi} (m0 + i u n0),
//   H1 = A r^{-1/2} e^{i phi} (-i) (m1 + i u n1),   u = XS/(k r),
// A = sqrt(2/(pi k)), times e^{-Im(k) r} for complex k.
template <bool CPLX, bool LOW>
__device__ __forceinline__ void hankel_asym(const WaveConst& W, double r, double rlo, double rinv, double sr, cd& h0,
                                            cd& h1)
{
    using A = Amp<LOW>;
    double sn, cs;
    sincos_phase<LOW>(W.kr, r, rlo, sn, cs);
    const double ri = rinv * A::SCALE;
    const double rho = ri * ri;
    if (!CPLX) {
        // w = (XS/(k r))^2 <= 1; its powers are shared by the four amplitude polynomials
        double p[A::N];
        p[1] = W.wr * rho;
#pragma unroll
        for (int m = 2; m < A::N; ++m) p[m] = p[m / 2] * p[m - m / 2];
        const double u = W.ur * ri;
        const double a = W.ampr * sr;
        const double er = cs * a, ei = sn * a;
        const double m1 = poly_pow<A::N>(A::m1, p), un1 = u * poly_pow<A::N>(A::n1, p);
        h1 = {fma(er, un1, ei * m1), fma(ei, un1, -er * m1)};
        const double m0 = poly_pow<A::N>(A::m0, p), un0 = u * poly_pow<A::N>(A::n0, p);
        h0 = {fma(er, m0, -ei * un0), fma(er, un0, ei * m0)};
    } else {
        const double x = W.wr * rho, y = W.wi * rho;
        const double R = 2.0 * x, S = fma(x, x, y * y);
        const cd u = {W.ur * ri, W.ui * ri};
        const double damp = exp(-W.ki * r) * sr;
        const cd e = cmul({cs * damp, sn * damp}, {W.ampr, W.ampi});
        cd m, n;
        poly_cplx_n<A::N>(A::m1, x, y, R, S, m.re, m.im);
        poly_cplx_n<A::N>(A::n1, x, y, R, S, n.re, n.im);
        const cd un1 = cmul(u, n);
        h1 = cmul(e, {m.im + un1.re, un1.im - m.re});
        poly_cplx_n<A::N>(A::m0, x, y, R, S, m.re, m.im);
        poly_cplx_n<A::N>(A::n0, x, y, R, S, n.re, n.im);
        const cd un0 = cmul(u, n);
        h0 = cmul(e, {m.re - un0.im, m.im + un0.re});
    }
}

// H0(k r) and H1(k r) when |k r| >= XS is known for the pair (no per-lane
// branch, no series), from the offset x - y = (rx + ex, ry + ey) and r2 = rx^2
// + ry^2; returns 1/r.
template <bool CPLX, bool LOW>
__device__ __forceinline__ double hankel01_far(const WaveConst& W, double rx, double ry, double ex, double ey,
                                               double r2, cd& h0, cd& h1)
{
    double r, rinv;
    sqrt_rsqrt(r2, r, rinv);
    hankel_asym<CPLX, LOW>(W, r, sqrt_error(rx, ry, ex, ey, r, rinv), rinv, rsqrt_nr(r), h0, h1);
    return rinv;
}

// The four entire functions of the series at t (N terms).
struct Entire {
    cd j0, e0, j1, e1;
};
template <bool CPLX, int N, int NTAB>
__device__ __forceinline__ Entire entire(const __attribute__((address_space(4))) SeriesTabs<NTAB>* c, double x, double y)
{
    Entire E;
    if (!CPLX) {
        E.j0.re = poly_n<N>(c->j0, x);
        E.e0.re = poly_n<N>(c->e0, x);
        E.j1.re = poly_n<N>(c->j1, x);
        E.e1.re = poly_n<N>(c->e1, x);
    } else {
        const double R = 2.0 * x, S = fma(x, x, y * y);
        poly_cplx_n<N>(c->j0, x, y, R, S, E.j0.re, E.j0.im);
        poly_cplx_n<N>(c->e0, x, y, R, S, E.e0.re, E.e0.im);
        poly_cplx_n<N>(c->j1, x, y, R, S, E.j1.re, E.j1.im);
        poly_cplx_n<N>(c->e1, x, y, R, S, E.e1.re, E.e1.im);
    }
    return E;
}

// H0(k r), H1(k r).  r2 = r^2, rinv = 1/r, srinv = r^{-1/2}, rlo as above.  Below XS the
// series, above it hankel_asym.
template <bool CPLX>
__device__ __forceinline__ void hankel01(const WaveConst& W, double r, double r2, double rinv, double srinv, cd& h0,
                                         cd& h1, double rlo = 0.0)
{
    const HankelTabsPtr T = hankel_tabs_fresh();
    constexpr double TWO_OVER_PI = 0.63661977236758134308;
    constexpr double EULER = 0.57721566490153286061;
    constexpr double LOW2 = (HANKEL_XS_F64 / SERIES_ZLOW) * (HANKEL_XS_F64 / SERIES_ZLOW);
    // both branches set these scalars and h0, h1 are written once after the
    // join: stores to different fields at the ends of the two branches would
    // be merged into one store through a selected address, which keeps the
    // caller's h0, h1 in scratch memory
    double h0r, h0i, h1r, h1i;
    if (r2 < W.r2_small) {
        const double lnr = log(r);
        Entire E;
        if (LOW2 * r2 < W.r2_small)
            E = entire<CPLX, SERIES_NLOW>(&T->low, W.tr * r2, W.ti * r2);
        else
            E = entire<CPLX, CPLX ? SERIES_NWIDE : SERIES_NMID>(&T->mid, fma(W.tr, r2, -SERIES_TMID), W.ti * r2);
        if (!CPLX) {
            const double zh = W.hr * r;
            const double j1 = zh * E.j1.re;
            const double lz = lnr + W.lkr;
            h0r = E.j0.re;
            h0i = fma(TWO_OVER_PI * (lz + EULER), E.j0.re, E.e0.re);
            h1r = j1;
            h1i = fma(W.y1r, rinv, fma(TWO_OVER_PI * lz, j1, zh * E.e1.re));
        } else {
            const cd zh = {W.hr * r, W.hi * r};
            const cd j1 = cmul(zh, E.j1);
            const cd lz = {lnr + W.lkr, W.lki};
            const cd y0 = cadd(cmul({TWO_OVER_PI * (lz.re + EULER), TWO_OVER_PI * lz.im}, E.j0), E.e0);
            const cd y1 = cadd(cadd(cscale({W.y1r, W.y1i}, rinv), cmul(cscale(lz, TWO_OVER_PI), j1)), cmul(zh, E.e1));
            h0r = E.j0.re - y0.im;
            h0i = E.j0.im + y0.re;
            h1r = j1.re - y1.im;
            h1i = j1.im + y1.re;
        }
    } else {
        cd a0, a1;
        hankel_asym<CPLX, false>(W, r, rlo, rinv, srinv, a0, a1);
        h0r = a0.re;
        h0i = a0.im;
        h1r = a1.re;
        h1i = a1.im;
    }
    h0 = {h0r, h0i};
    h1 = {h1r, h1i};
}

}  // namespace bemk
