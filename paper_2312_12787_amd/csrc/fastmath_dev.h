// fastmath_dev.h -- FP64 square roots and sine/cosine for the assembly's
// large-argument path (distances between distinct boundary points, phases
// k r of moderate size).  Built from the hardware reciprocal-square-root
// estimate and fused multiply-adds only: no IEEE special-case fix-ups, no
// table lookups, every constant a compile-time literal.
//
// Domains: sqrt_rsqrt / rsqrt_nr take normal x > 0; sincos_phase takes
// k r < 2^30 (the reduction below is exact there).
#pragma once

#include <hip/hip_runtime.h>

namespace bemk {

// r = sqrt(x) and ri = 1/sqrt(x): the v_rsq_f64 estimate y0 refined by two
// steps of Goldschmidt's coupled iteration, g -> sqrt(x), h -> 1/(2 sqrt(x)):
//   e = 1/2 - g h,  g <- g + g e,  h <- h + h e
// (quadratic convergence: a relative error eps of y0 leaves about eps^4).
__device__ __forceinline__ void sqrt_rsqrt(double x, double& r, double& ri)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    r = g;
    ri = h + h;
}

// 1/sqrt(x): the v_rsq_f64 estimate refined by two Newton steps for
// f(y) = 1/y^2 - x,  y <- y + (y/2)(1 - x y^2).
__device__ __forceinline__ double rsqrt_nr(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    return y;
}

// a - b = s + diff_error(a, b, s) exactly, s = a - b rounded (Knuth's two-sum).
__device__ __forceinline__ double diff_error(double a, double b, double s)
{
    const double bv = a - s;
    return (a - (s + bv)) + (bv - b);
}

// What r lacks of the distance sqrt((rx + ex)^2 + (ry + ey)^2), r being about
// sqrt(rx^2 + ry^2) and rinv 1/r:  (rx^2 + ry^2 - r^2 + 2 rx ex + 2 ry ey) / (2r),
// the squares of the larger component and of r subtracted first (they cancel)
// with the larger one's rounding kept.  Leaves about a tenth of an ulp of r.
__device__ __forceinline__ double sqrt_error(double rx, double ry, double ex, double ey, double r, double rinv)
{
    const double hi = fmax(fabs(rx), fabs(ry)), lo = fmin(fabs(rx), fabs(ry));
    const double hh = hi * hi;
    const double d = fma(lo, lo, fma(-r, r, hh)) + fma(hi, hi, -hh);
    return rinv * fma(0.5, d, fma(rx, ex, ry * ey));
}

// sin and cos of n pi/2 + t, n an integer, |t| <= pi/4 (+ rounding): Taylor
// series (LOW: to about 1e-10 instead of an ulp)
//   sin t = t - t^3/3! + ... - t^15/15! + t^17/17!   (truncation < 1e-19; LOW: t^11, 7e-12)
//   cos t = 1 - t^2/2! + ... + t^16/16!              (truncation < 3e-18; LOW: t^12, 4e-13)
// in u = t^2, then the quadrant n mod 4 swaps and negates.
template <bool LOW>
__device__ __forceinline__ void sincos_quadrant(double n, double t, double& s, double& c)
{
    const double u = t * t;
    // (-1)^m / (2m+1)! and (-1)^m / (2m)! (factorials exact in double)
    double ps, pc;
    if (LOW) {
        ps = -1.0 / 39916800.0;
        pc = 1.0 / 479001600.0;
    } else {
        ps = 1.0 / 355687428096000.0;             // 1/17!
        ps = fma(ps, u, -1.0 / 1307674368000.0);  // 1/15!
        ps = fma(ps, u, 1.0 / 6227020800.0);      // 1/13!
        ps = fma(ps, u, -1.0 / 39916800.0);       // 1/11!
        pc = 1.0 / 20922789888000.0;              // 1/16!
        pc = fma(pc, u, -1.0 / 87178291200.0);    // 1/14!
        pc = fma(pc, u, 1.0 / 479001600.0);       // 1/12!
    }
    ps = fma(ps, u, 1.0 / 362880.0);  // 1/9!
    ps = fma(ps, u, -1.0 / 5040.0);   // 1/7!
    ps = fma(ps, u, 1.0 / 120.0);     // 1/5!
    ps = fma(ps, u, -1.0 / 6.0);      // 1/3!
    pc = fma(pc, u, -1.0 / 3628800.0);  // 1/10!
    pc = fma(pc, u, 1.0 / 40320.0);     // 1/8!
    pc = fma(pc, u, -1.0 / 720.0);      // 1/6!
    pc = fma(pc, u, 1.0 / 24.0);        // 1/4!
    pc = fma(pc, u, -0.5);              // 1/2!
    const double st = fma(t * u, ps, t);
    const double ct = fma(u, pc, 1.0);
    // q = n mod 4;  sin = (q odd ? cos t : sin t) (-1)^[q in {2,3}],
    //                                       cos = (q odd ? sin t : cos t) (-1)^[q in {1,2}]
    // (two's complement: the low bits of a negative n are n mod 4 as well)
    const unsigned q = (unsigned)(int)n;
    const double a = (q & 1u) ? ct : st;
    const double b = (q & 1u) ? st : ct;
    s = __hiloint2double((int)((unsigned)__double2hiint(a) ^ ((q & 2u) << 30)), __double2loint(a));
    c = __hiloint2double((int)((unsigned)__double2hiint(b) ^ (((q + 1u) & 2u) << 30)), __double2loint(b));
}

// sin and cos of k (r + rlo) - pi/4, 0 < k r < 2^30.  The product k r is kept to twice the precision, so the
// phase is as good as r + rlo.  Cody and Waite's additive reduction x = k r =
// (n + 1/2) pi/2 + t, the -pi/4 of the Hankel functions being the 1/2, with
// pi/2 split into P1 = pi/2 rounded to double and P2 = pi/2 - P1 rounded: with
// a fused multiply-add, x - (n + 1/2) P1 is exact, and (n + 1/2) P2 leaves an
// error of about n 1.5e-33.
template <bool LOW>
__device__ __forceinline__ void sincos_phase(double k, double r, double rlo, double& s, double& c)
{
    constexpr double TWO_OVER_PI = 0x1.45f306dc9c883p-1;  // 2/pi
    constexpr double P1 = 0x1.921fb54442d18p+0;           // pi/2 rounded to double
    constexpr double P2 = 0x1.1a62633145c07p-54;          // pi/2 - P1 rounded to double
    const double x = k * r;
    const double n = rint(fma(x, TWO_OVER_PI, -0.5));
    const double nh = n + 0.5;
    const double e = fma(k, rlo, fma(k, r, -x));
    const double t = fma(-nh, P1, x) + fma(-nh, P2, e);
    sincos_quadrant<LOW>(n, t, s, c);
}

// sin and cos of x: the same reduction and series for |x| < 2^29; BIG: any x
// (the library's beyond 2^29).
template <bool BIG>
__device__ __forceinline__ void sincos_phase_any(double x, double& s, double& c)
{
    if (!BIG || fabs(x) < 0x1p29) {
        const double n = rint(x * 0x1.45f306dc9c883p-1);
        sincos_quadrant<false>(n, fma(-n, 0x1.1a62633145c07p-54, fma(-n, 0x1.921fb54442d18p+0, x)), s, c);
    } else {
        sincos(x, &s, &c);
    }
}

// sin(a) / a: the Taylor series to a^16 / 17! below 1/2 (truncation 2e-22)
template <bool BIG>
__device__ __forceinline__ double sinc(double a)
{
    if (fabs(a) > 0.5) {
        double s, c;
        sincos_phase_any<BIG>(a, s, c);
        return s / a;
    }
    const double u = a * a;
    double p = 1.0 / 355687428096000.0;     // 1/17!
    p = fma(p, u, -1.0 / 1307674368000.0);  // 1/15!
    p = fma(p, u, 1.0 / 6227020800.0);      // 1/13!
    p = fma(p, u, -1.0 / 39916800.0);       // 1/11!
    p = fma(p, u, 1.0 / 362880.0);          // 1/9!
    p = fma(p, u, -1.0 / 5040.0);           // 1/7!
    p = fma(p, u, 1.0 / 120.0);             // 1/5!
    p = fma(p, u, -1.0 / 6.0);              // 1/3!
    return fma(p, u, 1.0);
}

}  // namespace bemk
