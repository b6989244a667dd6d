// expansion_dev.h -- the sums of an element's Gauss rule against a point from
// ONE evaluation of H0 and H1, at the element's midpoint.  With x the point,
// c_j the midpoint, t_j and n_j the element's tangent and normal, r = |x - c_j|,
// phi the angle of x - c_j to t_j, s the position on the element, Graf's
// addition theorem gives
//   H0(k |x - c_j - s t_j|) = sum_{m in Z} J_m(k s) H_m(k r) cos(m phi),   |s| < r,
// so that the rule's sums, whatever its order, are
//   sum_g w_g H0                 = sum_{m even} mu_m H_m cos m phi,   mu_m = sum_g w_g J_m(k s_g)
//   sum_g w_g H1 (r_g.t_j)/r_g   = sum_{p odd > 0} (mu_{p-1} - mu_{p+1}) H_p cos p phi
//   sum_g w_g H1 (r_g.n_j)/r_g   = sum_{p odd > 0} (mu_{p-1} + mu_{p+1}) H_p sin p phi
// (odd moments vanish, the rule is symmetric; the two vector sums are -1/k
// times the gradient of the first), and with nu_m = 2 J_m(k h/2) the
// components along t_j and n_j of the end-point difference are
//   sum_{p even >= 0} (nu_{p-1} - nu_{p+1}) H_p cos p phi   (p = 0: -nu_1 H_0)
//   sum_{p even > 0}  (nu_{p-1} + nu_{p+1}) H_p sin p phi
// without the cancellation of the two end values.  H_2, H_3, ... follow by
// the upward recurrence (stable: it follows the growing solution), cos m phi
// and sin m phi by the Chebyshev recurrence.  The coefficients are a record
// per (side, element), made with the geometry tables.  Orders up to L leave a
// relative remainder of (h/(2r))^L (and (kh/4)^L/(L+1)! for large r); each
// record holds the distances beyond which L = 8, 10, 12, 16 and 20 leave less
// than 4e-17 (real k; internal.h).
#pragma once

#include "hankel_dev.h"
#include "internal.h"

namespace bemk {

typedef const __attribute__((address_space(4))) double* ScalarPtr;  // wave-uniform addresses: scalar loads

// The sums of one (point, element) pair without their i/4, i k/4 factors.
struct PairSums {
    cd S;       // sum w H0
    cd Gt, Gn;  // sum w H1 r/|r| along t_j and n_j
    cd Tt, Tn;  // end-point difference along t_j and n_j
};

__device__ __forceinline__ void add_scaled(cd& s, double c, double f, cd v)
{
    const double w = c * f;
    s.re = fma(w, v.re, s.re);
    s.im = fma(w, v.im, s.im);
}
__device__ __forceinline__ void add_scaled(cd& s, cd c, double f, cd v)
{
    const cd w = {c.re * f, c.im * f};
    s.re = fma(w.re, v.re, fma(-w.im, v.im, s.re));
    s.im = fma(w.re, v.im, fma(w.im, v.re, s.im));
}

// coefficient i of a record (cw doubles each: 2 where some domain of the
// problem is lossy)
template <bool CPLX>
struct Coef;
template <>
struct Coef<false> {
    template <class Ptr>
    static __device__ __forceinline__ double get(Ptr c, int cw, int i)
    {
        return c[cw * i];
    }
};
template <>
struct Coef<true> {
    template <class Ptr>
    static __device__ __forceinline__ cd get(Ptr c, int, int i)
    {
        return {c[2 * i], c[2 * i + 1]};
    }
};

// The expansion up to order Lo (even, >= BASE, uniform over the wave; orders
// up to BASE are unrolled): hz = H0, h1 = H1 at the midpoint distance, c1, s1
// = cos phi, sin phi, tz = 2/(k r).  VEC = false leaves out what only the
// Burton-Miller rows need: Gt, Tt and Tn.
template <bool CPLX, bool VEC, int BASE, class Ptr>
__device__ __forceinline__ PairSums expand(Ptr c, int cw, int Lo, cd hz, cd h1, double c1, double s1, cd tz)
{
    using K = Coef<CPLX>;
    PairSums P;
    P.S = P.Gt = P.Gn = P.Tt = P.Tn = {0.0, 0.0};
    add_scaled(P.S, K::get(c, cw, 0), 1.0, hz);
    if (VEC) add_scaled(P.Tt, K::get(c, cw, 1), 1.0, hz);
    cd Hp = hz, H = h1, q = {0.0, 0.0};
    double cp = 1.0, cc = c1, sp = 0.0, ss = s1;
    const double c2 = c1 + c1;
    auto next = [&]() {  // order m -> m + 1
        q.re += tz.re;
        if (CPLX) q.im += tz.im;  // q = m tz
        cd Hn;
        if (CPLX)
            Hn = {fma(q.re, H.re, fma(-q.im, H.im, -Hp.re)), fma(q.re, H.im, fma(q.im, H.re, -Hp.im))};
        else
            Hn = {fma(q.re, H.re, -Hp.re), fma(q.re, H.im, -Hp.im)};
        Hp = H;
        H = Hn;
        const double cn = fma(c2, cc, -cp), sn = fma(c2, ss, -sp);
        cp = cc;
        cc = cn;
        sp = ss;
        ss = sn;
    };
    auto two = [&](int p) {  // orders p (odd) and p + 1
        const int o = exp_pos(p);
        if (VEC) add_scaled(P.Gt, K::get(c, cw, o), cc, H);
        add_scaled(P.Gn, K::get(c, cw, o + 1), ss, H);
        next();
        add_scaled(P.S, K::get(c, cw, o + 2), cc, H);
        if (VEC) {
            add_scaled(P.Tt, K::get(c, cw, o + 3), cc, H);
            add_scaled(P.Tn, K::get(c, cw, o + 4), ss, H);
        }
    };
    two(1);
#pragma unroll
    for (int p = 3; p < BASE; p += 2) {
        next();
        two(p);
    }
    for (int p = BASE + 1; p < Lo; p += 2) {
        next();
        two(p);
    }
    return P;
}

}  // namespace bemk
