// assemble.hip -- setup kernels (element table, Gauss rule, per-domain
// constants, self terms) and the fused assembly of the collocation matrix
// of the Calderon-ordered Burton-Miller system (Secs. 3-7 of arXiv 2312.12787).
#include <hip/hip_runtime.h>

#include "expansion_dev.h"
#include "gauss_tables.h"
#include "hankel_dev.h"
#include "hankel_tables.h"
#include "internal.h"
#include "launch.h"

namespace bemk {

namespace {

constexpr double PI = 3.14159265358979323846;
constexpr double EULER = 0.57721566490153286061;
template <class T>
__device__ __forceinline__ const T* tab(const char* g, size_t off) { return reinterpret_cast<const T*>(g + off); }
template <class T>
__device__ __forceinline__ T* tabw(char* g, size_t off) { return reinterpret_cast<T*>(g + off); }

__device__ __forceinline__ cd cdiv(cd a, cd b)
{
    const double den = b.re * b.re + b.im * b.im;
    return {(a.re * b.re + a.im * b.im) / den, (a.im * b.re - a.re * b.im) / den};
}
__device__ __forceinline__ cd csqrt_(cd z)
{
    const double r = hypot(z.re, z.im);
    double sr = sqrt(0.5 * (r + fabs(z.re)));
    if (sr == 0.0) return {0.0, 0.0};
    if (z.re >= 0.0) return {sr, z.im / (2.0 * sr)};
    return {fabs(z.im) / (2.0 * sr), z.im >= 0.0 ? sr : -sr};
}
__device__ __forceinline__ cd clog_(cd z) { return {log(hypot(z.re, z.im)), atan2(z.im, z.re)}; }

// Squared distance beyond which an expansion order with the limits x and kamax
// serves an element of half length a at |k| = ak (internal.h); infinite if none.
__device__ __forceinline__ double expansion_limit(double a, double ak, double x, double kamax)
{
    const double ka = ak * a, v = a / x;
    return ka >= EXP_KA_MIN && ka <= kamax ? v * v : __longlong_as_double(0x7ff0000000000000ll);
}

__device__ __forceinline__ bool expanded(double close2) { return close2 < __longlong_as_double(0x7ff0000000000000ll); }

// ---------------------------------------------------------------------------
// Element table (Secs. 4, 7).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void setup_element(char* g, const GeomLayout& L, int e)
{
    const double2* nodes = tab<double2>(g, L.nodes);
    const int2 ab = tab<int2>(g, L.elnodes)[e];
    const double2 a = nodes[ab.x], b = nodes[ab.y];
    ElemRec E;
    E.ax = a.x;
    E.ay = a.y;
    E.bx = b.x;
    E.by = b.y;
    E.cx = 0.5 * (a.x + b.x);
    E.cy = 0.5 * (a.y + b.y);
    const double dx = b.x - a.x, dy = b.y - a.y;
    E.h = sqrt(dx * dx + dy * dy);
    E.tx = dx / E.h;
    E.ty = dy / E.h;
    E.nx = -E.ty;
    E.ny = E.tx;
    for (int k = 0; k < 3; ++k) E.pad[k] = 0.0;
    const IfacePlan P = tab<IfacePlan>(g, L.iface)[tab<int>(g, L.elif)[e]];
    const DomIn* in = tab<DomIn>(g, L.dom_in);
    for (int side = 0; side < 2; ++side) {
        const int d = side ? P.dr : P.dl;
        const double lim = expansion_limit(0.5 * E.h, hypot(in[d].k[0], in[d].k[1]), EXP_X20, EXP_KA_MAX);
        E.close2[side] = expanded(lim) ? lim : 6.25 * E.h * E.h;
    }
    tabw<ElemRec>(g, L.elem)[e] = E;
}

// ---------------------------------------------------------------------------
// Per-domain constants: eps_d = (k_d/k_0)^2 (Sec. 2), the Burton-Miller
// coefficient alpha/eps_d (Sec. 6 recipe), the row scaling beta (Sec. 5) and
// the Hankel tables of the wavenumber.
// ---------------------------------------------------------------------------
__device__ void build_wave(cd k, WaveConst& W)
{
    const double ak = hypot(k.re, k.im);
    W.kr = k.re;
    W.ki = k.im;
    const double rs = series_radius(k.re, k.im) / ak;
    W.r2_small = rs * rs;
    const cd xk = cdiv({HANKEL_XS_F64, 0.0}, k);  // XS / k
    W.ur = xk.re;
    W.ui = xk.im;
    const cd w = cmul(xk, xk);
    W.wr = w.re;
    W.wi = w.im;
    const cd sq = csqrt_(cdiv({2.0 / PI, 0.0}, k));  // sqrt(2/(pi k))
    W.ampr = sq.re;
    W.ampi = sq.im;
    const cd tk = cdiv({2.0, 0.0}, k);
    W.tkr = tk.re;
    W.tki = tk.im;
    const cd h = cscale(k, 0.5);
    W.hr = h.re;
    W.hi = h.im;
    const cd t = cmul(h, h);
    W.tr = t.re;
    W.ti = t.im;
    const cd lk = clog_(h);
    W.lkr = lk.re;
    W.lki = lk.im;
    const cd y1 = cdiv({-2.0 / PI, 0.0}, k);
    W.y1r = y1.re;
    W.y1i = y1.im;
}

__device__ __forceinline__ void setup_domain(char* g, const GeomLayout& L, int d)
{
    const GlobalIn G = *tab<GlobalIn>(g, L.glob_in);
    if (d >= G.n_dom) return;
    const DomIn* in = tab<DomIn>(g, L.dom_in);
    const cd k0 = {in[0].k[0], in[0].k[1]};
    const cd k = {in[d].k[0], in[d].k[1]};
    const cd r = cdiv(k, k0);
    const cd eps = cmul(r, r);
    // alpha = -i / k0 (Sec. 3.3) unless given
    const cd alpha = G.has_alpha ? cd{G.alpha[0], G.alpha[1]} : cdiv({0.0, -1.0}, k0);
    cd beta;
    if (G.has_beta)
        beta = {G.beta[0], G.beta[1]};
    else if (G.form == 0 || G.form == 3)
        beta = {-alpha.re, -alpha.im};
    else
        beta = {1.0, 0.0};
    const cd c = in[d].has_bm ? cd{in[d].bm[0], in[d].bm[1]} : cdiv(alpha, eps);
    DomConst D;
    D.k[0] = k.re;
    D.k[1] = k.im;
    D.eps[0] = eps.re;
    D.eps[1] = eps.im;
    D.c[0] = c.re;
    D.c[1] = c.im;
    D.beta[0] = beta.re;
    D.beta[1] = beta.im;
    D.cplx = (k.im != 0.0);
    D.pad = 0;
    tabw<DomConst>(g, L.dom)[d] = D;
    build_wave(k, tabw<WaveConst>(g, L.wave)[d]);
}

// ---------------------------------------------------------------------------
// Self term of the single-layer operator on a flat element at its midpoint
// (Sec. 7, the weak singularity): S_ii = (i/(2k)) int_0^{kh/2} H0(t) dt, the
// integral taken term by term from the ascending series of J0 and Y0 (long
// elements: int_h0_long).
// One lane per (element, domain on either side of it).
// ---------------------------------------------------------------------------
__device__ cd int_h0(cd z)
{
    const cd zh = cscale(z, 0.5);
    const cd q = cmul(zh, zh);
    const cd lz = clog_(zh);
    cd T = cscale(zh, 2.0);  // 2 (z/2)^{2m+1} (-1)^m / (m!)^2
    cd sj = {0.0, 0.0}, sj2 = {0.0, 0.0}, sh = {0.0, 0.0};
    double hm = 0.0;
    for (int m = 0; m < 200; ++m) {
        if (m > 0) {
            T = cscale(cmul(T, q), -1.0 / ((double)m * m));
            hm += 1.0 / m;
        }
        const double o = 2.0 * m + 1.0;
        const cd a = cscale(T, 1.0 / o);
        sj = cadd(sj, a);
        sj2 = cadd(sj2, cscale(T, 1.0 / (o * o)));
        sh = cadd(sh, cscale(a, hm));
        if (m > 3 && fabs(a.re) + fabs(a.im) < 1e-18 * (fabs(sj.re) + fabs(sj.im))) break;
    }
    // int Y0 = (2/pi) [ (ln(z/2) + gamma) sum T/(2m+1) - sum T/(2m+1)^2 - sum H_m T/(2m+1) ]
    const cd ly = cmul({lz.re + EULER, lz.im}, sj);
    const cd iy = cscale({ly.re - sj2.re - sh.re, ly.im - sj2.im - sh.im}, 2.0 / PI);
    return {sj.re - iy.im, sj.im + iy.re};  // int J0 + i int Y0
}

// The same for |z| > 4, which only elements longer than 1.2 wavelengths reach and
// where the series loses digits to cancellation (|z| = 6: 3e-15, 14: 3e-12).  Up
// to |z| = 40 the rest of the ray in steps of at most 2 by the 16-point rule.
// Beyond, from int_0^inf H0 = 1, 1 minus the integral of the asymptotic form
//   H0(t) = sqrt(2/(pi t)) e^{i(t - pi/4)} sum_m c_m t^{-m},  c_m = c_{m-1} (2m - 1)^2 / (8 i m),
// term by term: its antiderivative that vanishes at i inf has, in place of c_m, d_m with
//   i d_m - (m - 1/2) d_{m-1} = c_m
// (the terms fall to about e^{-|z|} before they grow).
__device__ cd int_h0_long(cd z)
{
    const double b = hypot(z.re, z.im);
    const cd e = cscale(z, 1.0 / b);
    if (b <= 40.0) {
        WaveConst W;
        build_wave(e, W);
        const int steps = (int)ceil(0.5 * (b - 4.0));
        const double half = 0.5 * (b - 4.0) / steps;
        cd sum = {0.0, 0.0};
        for (int i = 0; i < 16 * steps; ++i) {
            const double r = 4.0 + half * (2 * (i / 16) + 1 + GAUSS_X[15][i % 16]);
            cd h0, h1;
            hankel01<true>(W, r, r * r, 1.0 / r, sqrt(1.0 / r), h0, h1);
            const double w = half * GAUSS_W[15][i % 16];
            sum = {fma(w, h0.re, sum.re), fma(w, h0.im, sum.im)};
        }
        return cadd(int_h0(cscale(e, 4.0)), cmul(e, sum));
    }
    const cd iz = cdiv({1.0, 0.0}, z);
    cd c = {1.0, 0.0}, d = {0.0, -1.0}, p = {1.0, 0.0}, sum = d;  // p = z^{-m}
    for (int m = 1; m <= 40; ++m) {
        const double f = (2.0 * m - 1.0) * (2.0 * m - 1.0) / (8.0 * m);
        c = {f * c.im, -f * c.re};
        const cd t = {fma(m - 0.5, d.re, c.re), fma(m - 0.5, d.im, c.im)};  // i d_m
        d = {t.im, -t.re};
        p = cmul(p, iz);
        sum = cadd(sum, cmul(d, p));
    }
    double sn, cs;
    sincos(z.re - 0.25 * PI, &sn, &cs);
    const cd amp = cmul(csqrt_(cscale(iz, 2.0 / PI)), cscale({cs, sn}, exp(-z.im)));
    return cadd({1.0, 0.0}, cmul(amp, sum));
}

__device__ __forceinline__ void setup_self(char* g, const GeomLayout& L, int N, int e, int side)
{
    const double2* nodes = tab<double2>(g, L.nodes);
    const int2 ab = tab<int2>(g, L.elnodes)[e];
    const IfacePlan P = tab<IfacePlan>(g, L.iface)[tab<int>(g, L.elif)[e]];
    const int d = side ? P.dr : P.dl;
    const DomIn* in = tab<DomIn>(g, L.dom_in);
    const cd k = {in[d].k[0], in[d].k[1]};
    const double dx = nodes[ab.y].x - nodes[ab.x].x, dy = nodes[ab.y].y - nodes[ab.x].y;
    const cd z = cscale(k, 0.5 * sqrt(dx * dx + dy * dy));
    const cd I = hypot(z.re, z.im) > 4.0 ? int_h0_long(z) : int_h0(z);
    const cd pre = cdiv({0.0, 0.5}, k);  // i / (2k)
    const cd s = cmul(pre, I);
    tabw<double2>(g, L.self)[(size_t)d * N + e] = make_double2(s.re, s.im);
}

// 1/n, n = 1 .. 47 (the series below multiply by them instead of dividing)
struct Reciprocals {
    double v[48];
};
constexpr Reciprocals make_reciprocals()
{
    Reciprocals r{};
    for (int n = 1; n < 48; ++n) r.v[n] = 1.0 / n;
    return r;
}
static __device__ const Reciprocals g_rcp = make_reciprocals();

// sum_j (-1)^j y^{2j+m} / (j! (m+j)!) W_{2j+m}: J_m(2 y) with W = 1 (mom null);
// with the moments W_n of the Gauss rule (n even: mom[n/2]) the rule's value
// of the integral of J_m(2 y x) over x in [-1, 1].  |y| <= EXP_KA_MAX / 2.
__device__ __forceinline__ cd bessel_sum(int m, cd y, const double* __restrict__ mom)
{
    cd t = {1.0, 0.0};
    for (int n = 1; n <= m; ++n) t = cscale(cmul(t, y), g_rcp.v[n]);
    const cd y2 = cmul(y, y);
    cd s = {0.0, 0.0};
    for (int j = 0; j < EXP_NTERMS; ++j) {
        const double w = mom ? mom[min(j + m / 2, GAUSS_NMOM - 1)] : 1.0;
        s.re = fma(t.re, w, s.re);
        s.im = fma(t.im, w, s.im);
        t = cscale(cmul(t, y2), -g_rcp.v[j + 1] * g_rcp.v[m + j + 1]);
    }
    return s;
}

// The expansion record of one element in the domain on one side of it, order m
// of it (and the head with order 0); see ExpHead.
__device__ __forceinline__ void setup_expansion(char* g, const GeomLayout& L, int N, int q, int e, int side, int m)
{
    const double2* nodes = tab<double2>(g, L.nodes);
    const int2 ab = tab<int2>(g, L.elnodes)[e];
    const IfacePlan P = tab<IfacePlan>(g, L.iface)[tab<int>(g, L.elif)[e]];
    const int d = side ? P.dr : P.dl;
    const DomIn* in = tab<DomIn>(g, L.dom_in);
    const cd k = {in[d].k[0], in[d].k[1]};
    const double dx = nodes[ab.y].x - nodes[ab.x].x, dy = nodes[ab.y].y - nodes[ab.x].y;
    const double a = 0.5 * sqrt(dx * dx + dy * dy);
    const double ak = hypot(k.re, k.im);
    const cd y = cscale(k, 0.5 * a);
    double* rec = tabw<double>(g, L.expn) + ((size_t)side * N + e) * L.exp_stride;
    if (m == 0) {
        auto sq = [](double v) { return v * v; };
        auto lim = [&](double x, double kamax) { return expansion_limit(a, ak, x, kamax); };
        ExpHead* H = reinterpret_cast<ExpHead*>(rec);
        H->close2 = lim(EXP_X20, EXP_KA_MAX);
        const double rs = series_radius(k.re, k.im) / ak;
        H->near64 = fmax(H->close2, sq(rs));
        H->lim8 = lim(EXP_X8, EXP_KA8);
        H->lim10 = lim(EXP_X10, EXP_KA10);
        H->lim12 = lim(EXP_X12, EXP_KA12);
        H->lim16 = lim(EXP_X16, EXP_KA16);
        H->near32 = fmax(lim(EXP32_X16, EXP_KA_MAX), sq(HANKEL_XS_F32 / ak));
        H->lim32_4 = lim(EXP32_X4, EXP32_KA4);
        H->lim32_6 = lim(EXP32_X6, EXP32_KA6);
        H->lim32_8 = lim(EXP32_X8, EXP32_KA8);
        H->take64 = expanded(H->close2) ? H->near64 : sq(rs + a);
        H->take32 = expanded(H->close2) ? H->near32 : sq(HANKEL_XS_F32 / ak + a);
    }
    const int cw = L.exp_cplx ? 2 : 1;  // doubles per coefficient
    double* c = rec + EXP_HEAD + cw * exp_pos(m);
    auto put = [&](int i, cd v) {
        c[cw * i] = v.re;
        if (cw == 2) c[cw * i + 1] = v.im;
    };
    const double* mom = GAUSS_MOM[q - 1];
    if (m & 1) {
        const cd u0 = cscale(bessel_sum(m - 1, y, mom), a), u1 = cscale(bessel_sum(m + 1, y, mom), a);
        put(0, {u0.re - u1.re, u0.im - u1.im});
        put(1, {u0.re + u1.re, u0.im + u1.im});
    } else {
        put(0, cscale(bessel_sum(m, y, mom), m ? 2.0 * a : a));
        const cd v1 = bessel_sum(m + 1, y, nullptr);
        if (m == 0) {
            put(1, cscale(v1, -2.0));
        } else {
            const cd v0 = bessel_sum(m - 1, y, nullptr);
            put(1, {2.0 * (v0.re - v1.re), 2.0 * (v0.im - v1.im)});
            put(2, {2.0 * (v0.re + v1.re), 2.0 * (v0.im + v1.im)});
        }
    }
}

// All device tables of a problem in one launch: they depend on the uploaded
// inputs alone (a lane forms the element length or the wavenumber it needs
// again), so nothing has to wait for another table.  Block 0 takes the
// domains and the Gauss rule, then come the elements, the self terms of both
// sides and the expansion records, one order of one record per lane.  Bound by
// one lane's chain of dependent operations, not by the work.  Measured with
// the assembly of 777 elements behind it: 346 us while four launches ran in
// turn (one of them, 39 us, a Newton iteration for the Gauss rule), 288 us
// with this one and the rule as a table.
constexpr int SETUP_BS = 64;
__global__ __launch_bounds__(SETUP_BS) void k_setup(char* g, GeomLayout L, int N, int n_dom, int q, int eblocks)
{
    int b = blockIdx.x;
    const int t = threadIdx.x;
    if (b == 0) {
        double* gl = tabw<double>(g, L.gl);
        if (t < QMAX) {
            gl[t] = GAUSS_X[q - 1][t];
            gl[QMAX + t] = GAUSS_W[q - 1][t];
        }
        if (t < n_dom) setup_domain(g, L, t);
        return;
    }
    b -= 1;
    const int part = b / eblocks, e = (b - part * eblocks) * SETUP_BS + t;
    if (e >= N) return;
    if (part == 0)
        setup_element(g, L, e);
    else if (part <= 2)
        setup_self(g, L, N, e, part - 1);
    else
        setup_expansion(g, L, N, q, e, (part - 3) & 1, (part - 3) >> 1);
}

// ---------------------------------------------------------------------------
// Fused assembly of one equation block (one side of an interface) against the
// elements of one interface.  Operators (eqs. (stmp)-(ddtmp)) of domain d
// between collocation point x_i and element j, by the q-point Gauss rule:
//   S  = (i/4)   sum_g w_g H0(k r_g)
//   D  = (ik/4)  sum_g w_g H1(k r_g) (r_g . n_j)/r_g
//   D* = -(ik/4) sum_g w_g H1(k r_g) (r_g . n_i)/r_g
//   N  = k^2 (n_i.n_j) S + (ik/4)[E(b_j) - E(a_j)],  E(p) = H1(k|x_i-p|) t_i.(x_i-p)/|x_i-p|
// (N by the identity d2G/dnx dny = k^2 (nx.ny) G - d2G/dtx dty, exact on a
// flat element).
// Block entries (sigma = +1 if the normal leaves domain d, eps = eps_d):
//   standard row, scale s:  A[row, u_j] = s (delta/2 + sigma D),   A[row, w_j] = -s sigma eps S
//   Burton-Miller row, c:   A[row, u_j] = delta/2 + sigma (D + c N),
//                           A[row, w_j] = -sigma eps S + c (eps delta/2 - sigma eps D*)
//
// All four sums come from ONE evaluation of H0 and H1, at the element's
// midpoint (expansion_dev.h).  Closer than a few element lengths, or for
// elements longer than about 0.8 wavelengths, the Gauss points are evaluated one
// by one.
// ---------------------------------------------------------------------------

// Per-block combination constants of one equation block (see the entries above).
struct BlockConst {
    cd cD, cS, cDs, cNS, cNE, du, dw, iq;
};

template <bool BM>
__device__ __forceinline__ BlockConst block_const(const DomConst& Dm, int sg)
{
    const cd k = {Dm.k[0], Dm.k[1]};
    const cd ik4 = {-0.25 * k.im, 0.25 * k.re};  // i k / 4
    const cd eps = {Dm.eps[0], Dm.eps[1]};
    const cd c = {Dm.c[0], Dm.c[1]};
    const cd beta = {Dm.beta[0], Dm.beta[1]};
    const double s = (double)sg;
    BlockConst B;
    B.iq = {0.0, 0.25};
    B.cD = BM ? cd{s * ik4.re, s * ik4.im} : cscale(cmul(beta, ik4), s);  // multiplies sum D
    B.cS = cscale(cmul(eps, B.iq), -s);                                   // multiplies sum S (w column)
    if (!BM) B.cS = cmul(B.cS, beta);
    B.cDs = cscale(cmul(cmul(c, eps), ik4), s);            // multiplies sum D* (the minus signs cancel)
    B.cNS = cscale(cmul(cmul(c, cmul(k, k)), B.iq), s);    // k^2 (n_i.n_j) S part of c sigma N
    B.cNE = cscale(cmul(c, ik4), s);                       // end-point part of c sigma N
    B.du = BM ? cd{0.5, 0.0} : cscale(beta, 0.5);          // jump term, u column
    B.dw = cscale(cmul(c, eps), 0.5);                      // jump term, w column (BM only)
    return B;
}

// Waves per SIMD that the far and near kernels leave room for.
constexpr int FAR_WAVES = 3, NEAR_WAVES = 2, ALL_WAVES = 3;

// Entries of the u and w columns from the sums (tt = t_i.t_j, tn = t_i.n_j;
// in the plane n_i.n_j = tt and n_i.t_j = -tn).
template <bool BM>
__device__ __forceinline__ void combine(const BlockConst& B, const PairSums& P, double tt, double tn, cd& au, cd& aw)
{
    au = cmul(B.cD, P.Gn);
    aw = cmul(B.cS, P.S);
    if (BM) {
        const cd Ds = {fma(tt, P.Gn.re, -tn * P.Gt.re), fma(tt, P.Gn.im, -tn * P.Gt.im)};
        const cd T = {fma(tt, P.Tt.re, tn * P.Tn.re), fma(tt, P.Tt.im, tn * P.Tn.im)};
        au = cadd(au, cadd(cscale(cmul(B.cNS, P.S), tt), cmul(B.cNE, T)));
        aw = cadd(aw, cmul(B.cDs, Ds));
    }
}

__device__ __forceinline__ void store_entry(double2* A, size_t lda, float2* A32, size_t row, int j, int N, cd au, cd aw)
{
    A[row + (size_t)j * lda] = make_double2(au.re, au.im);
    A[row + (size_t)(N + j) * lda] = make_double2(aw.re, aw.im);
    if (A32) {
        A32[row + (size_t)j * lda] = make_float2((float)au.re, (float)au.im);
        A32[row + (size_t)(N + j) * lda] = make_float2((float)aw.re, (float)aw.im);
    }
}
__device__ __forceinline__ void store_entry(float2* A, size_t lda, float2*, size_t row, int j, int N, cd au, cd aw)
{
    A[row + (size_t)j * lda] = make_float2((float)au.re, (float)au.im);
    A[row + (size_t)(N + j) * lda] = make_float2((float)aw.re, (float)aw.im);
}

// Squared distance of a collocation point and a midpoint.  The far and the
// near launch compare it, formed by the same operations, with the same limit,
// so each element of a wave is taken by exactly one of them.
__device__ __forceinline__ double pair_r2(double rx, double ry) { return fma(rx, rx, ry * ry); }

// Element records through scalar loads: position of each field in ElemRec
constexpr int E_CX = 0, E_CY = 1, E_TX = 2, E_TY = 3;
static_assert(offsetof(ElemRec, cx) == 0 && offsetof(ElemRec, tx) == 16 && offsetof(ElemRec, nx) == 32,
              "scalar reads of the element records");

// A table entry at a wave-uniform address, read by scalar loads once (stores
// to the matrix do not make the compiler read it again).
template <class T>
__device__ __forceinline__ T scalar_copy(const T* p)
{
    static_assert(sizeof(T) % sizeof(double) == 0, "copied as doubles");
    T out;
    ScalarPtr src = (ScalarPtr)p;
    double* dst = reinterpret_cast<double*>(&out);
#pragma unroll
    for (size_t k = 0; k < sizeof(T) / sizeof(double); ++k) dst[k] = src[k];
    return out;
}

// What a launch needs besides its rows.
template <class T2>
struct AsmArgs {
    const char* g;
    GeomLayout L;
    int N, n_if, q;
    T2* A;
    float2* A32;  // FP32 copy of an FP64 matrix, or null
    size_t lda;
    bool point_launch;  // elements without expansion have a launch of their own
};

// ---------------------------------------------------------------------------
// Far launch: every element whose midpoint is, for all rows of the wave, at
// least XS/|k| away and within reach of the expansion.  One lane per row, one
// wave per (64 rows, `per` elements of a column chunk); the element's data are
// wave-uniform (scalar loads), so there is no LDS and no barrier, and a wave
// skips the elements that the near launch takes by one ballot.
// Bound by FP64 VALU issue: about 360 instructions per pair of a
// Burton-Miller row and 270 of a standard row (real k, FP64), of which the
// Hankel evaluation is 150 (point by point the q-point rule took q + 1 of
// them).  Distance, phase and recurrences are FP64 in the FP32 assembly too
// (an FP64 FMA issues as fast as an FP32 one); that path takes the shorter
// amplitude polynomials and fewer orders.  Measured, geometry tables and
// assembly, against point-by-point sums: kite of 4096 elements, one lossy
// wavenumber, 2019 -> 645 us; 8192 elements in FP32 3280 -> 1106 us, the
// entries' error against 32-digit values 2 to 5 times smaller; 777 elements at
// k h = 0.8 288 -> 68 us (50 in the single launch below); three sectors,
// 1900 elements, 1005 -> 185 us (154).
// Entries in FP64 are as close to 32-digit values as point-by-point sums, which
// averaged the rounding of q evaluations (standard rows, w columns, rms: disk of
// 256 elements 2.2e-16 both, kite of 512 6.9e-16 -> 5.2e-16, of 300 at arg k = 5.7
// degrees 3.2e-15 -> 7.0e-16): the phase k r is formed from a compensated
// distance, the series below |k r| = 6 do not cancel (hankel_dev.h).
// ---------------------------------------------------------------------------
template <bool CPLX, bool BM, class T2>
__device__ __forceinline__ void far_part(const AsmArgs<T2>& P, int side, int tile, int li, int col_part, int per)
{
    constexpr bool LOW = sizeof(T2) == sizeof(float2);
    constexpr int BASE = LOW ? 4 : 8;
    const Tile rt = tab<Tile>(P.g, P.L.rtiles)[tile];
    const int parts = COL_CHUNK / per;
    const Tile cc = tab<Tile>(P.g, P.L.cchunks)[col_part / parts];
    const int j0 = col_part % parts * per;
    const int j1 = min(j0 + per, cc.count);
    if (li >= rt.count || j0 >= j1) return;
    const IfacePlan F = tab<IfacePlan>(P.g, P.L.iface)[rt.iface];
    const int d = side ? F.dr : F.dl;
    const int sg = tab<int>(P.g, P.L.sigma)[d * P.n_if + cc.iface];
    const int i = rt.start + li;
    const size_t row = (size_t)((side ? F.row_r : F.row_l) + (i - F.off));
    if (sg == 0) {  // this domain does not touch the interface
        for (int jj = j0; jj < j1; ++jj) store_entry(P.A, P.lda, P.A32, row, cc.start + jj, P.N, {0.0, 0.0}, {0.0, 0.0});
        return;
    }
    // the record of an element holds both of its sides: take the one in domain d
    const int jside = tab<IfacePlan>(P.g, P.L.iface)[cc.iface].dr == d ? 1 : 0;
    const WaveConst W = scalar_copy(tab<WaveConst>(P.g, P.L.wave) + d);
    const BlockConst B = block_const<BM>(tab<DomConst>(P.g, P.L.dom)[d], sg);
    const ElemRec* Ei = tab<ElemRec>(P.g, P.L.elem) + i;
    const double xi = Ei->cx, yi = Ei->cy, tix = Ei->tx, tiy = Ei->ty;
    const cd tk = {W.tkr, W.tki};
    const int cw = P.L.exp_cplx ? 2 : 1;
    for (int jj = j0; jj < j1; ++jj) {
        const int j = cc.start + jj;
        ScalarPtr Ej = (ScalarPtr)(tab<ElemRec>(P.g, P.L.elem) + j);
        ScalarPtr rec = (ScalarPtr)(tab<double>(P.g, P.L.expn) + ((size_t)jside * P.N + j) * P.L.exp_stride);
        const double cx = Ej[E_CX], cy = Ej[E_CY], tx = Ej[E_TX], ty = Ej[E_TY];
        const double rx = xi - cx, ry = yi - cy;
        const double r2 = pair_r2(rx, ry);
        auto closer = [&](double lim2) { return __builtin_amdgcn_ballot_w64(r2 < lim2) != 0; };
        if (closer(rec[LOW ? EXP_H_NEAR32 : EXP_H_NEAR64])) continue;
        int Lo = BASE;
        if (LOW) {
            if (closer(rec[EXP_H_LIM32]))
                Lo = !closer(rec[EXP_H_LIM32 + 1]) ? 6 : !closer(rec[EXP_H_LIM32 + 2]) ? 8 : 16;
        } else if (closer(rec[EXP_H_LIM])) {
            Lo = !closer(rec[EXP_H_LIM + 1]) ? 10 : !closer(rec[EXP_H_LIM + 2]) ? 12 : !closer(rec[EXP_H_LIM + 3]) ? 16 : 20;
        }
        // the rounding of the two differences, for the phase
        const double ex = diff_error(xi, cx, rx), ey = diff_error(yi, cy, ry);
        cd h0, h1;
        const double rinv = hankel01_far<CPLX, LOW>(W, rx, ry, ex, ey, r2, h0, h1);
        const double c1 = fma(rx, tx, ry * ty) * rinv, s1 = fma(ry, tx, -rx * ty) * rinv;
        const PairSums sums =
            expand<CPLX, BM, BASE>(rec + EXP_HEAD, cw, Lo, h0, h1, c1, s1, {tk.re * rinv, CPLX ? tk.im * rinv : 0.0});
        cd au, aw;
        combine<BM>(B, sums, fma(tix, tx, tiy * ty), fma(tiy, tx, -tix * ty), au, aw);
        store_entry(P.A, P.lda, P.A32, row, j, P.N, au, aw);
    }
}
template <bool CPLX, bool BM, class T2>
__global__ __launch_bounds__(ROW_TILE, FAR_WAVES) void k_assemble_far(const AsmArgs<T2> P, int side,
                                                                      const int* __restrict__ tiles, int per)
{
    far_part<CPLX, BM>(P, side, tiles[blockIdx.x], threadIdx.x, blockIdx.y, per);
}

// ---------------------------------------------------------------------------
// Elements without expansion (|k| h/2 beyond EXP_KA_MAX or below EXP_KA_MIN),
// for rows whose points are all at least XS/|k| from theirs: point by point, one
// lane per row, over the far launch's grid; launched only where a domain has such
// elements (a good conductor's |k| is large against any mesh of the host).  An
// end point's value serves both elements that meet there.  Bound by FP64 VALU
// issue, q + 1 Hankel evaluations per pair.  As "close" pairs of the near launch,
// an LDS round per 3 to 6 of them, 4096 elements at |k| h/2 = 4 took 3.81 ms in
// FP64 and in FP32, now 1.93 and 1.31.
// ---------------------------------------------------------------------------
template <bool CPLX, bool BM, class T2>
__global__ __launch_bounds__(ROW_TILE, NEAR_WAVES) void k_assemble_points(const AsmArgs<T2> P, int side,
                                                                          const int* __restrict__ tiles, int per)
{
    constexpr bool LOW = sizeof(T2) == sizeof(float2);
    const Tile rt = tab<Tile>(P.g, P.L.rtiles)[tiles[blockIdx.x]];
    const int parts = COL_CHUNK / per, li = threadIdx.x;
    const Tile cc = tab<Tile>(P.g, P.L.cchunks)[blockIdx.y / parts];
    const int j0 = blockIdx.y % parts * per, j1 = min(j0 + per, cc.count);
    if (li >= rt.count || j0 >= j1) return;
    const IfacePlan F = tab<IfacePlan>(P.g, P.L.iface)[rt.iface];
    const int d = side ? F.dr : F.dl;
    const int sg = tab<int>(P.g, P.L.sigma)[d * P.n_if + cc.iface];
    if (sg == 0) return;
    const int i = rt.start + li;
    const size_t row = (size_t)((side ? F.row_r : F.row_l) + (i - F.off));
    const int jside = tab<IfacePlan>(P.g, P.L.iface)[cc.iface].dr == d ? 1 : 0;
    const WaveConst W = scalar_copy(tab<WaveConst>(P.g, P.L.wave) + d);
    const BlockConst B = block_const<BM>(tab<DomConst>(P.g, P.L.dom)[d], sg);
    const ElemRec* Ei = tab<ElemRec>(P.g, P.L.elem) + i;
    const double xi = Ei->cx, yi = Ei->cy, tix = Ei->tx, tiy = Ei->ty;
    ScalarPtr gl = (ScalarPtr)tab<double>(P.g, P.L.gl);
    auto hankel = [&](double rx, double ry, cd& h0, cd& h1) {
        double r, rinv;
        sqrt_rsqrt(fma(rx, rx, ry * ry), r, rinv);
        hankel_asym<CPLX, LOW>(W, r, 0.0, rinv, rsqrt_nr(r), h0, h1);
        return rinv;
    };
    auto end_value = [&](double px, double py) {
        const double rx = xi - px, ry = yi - py;
        cd h0, h1;
        const double rinv = hankel(rx, ry, h0, h1);
        return cscale(h1, fma(rx, tix, ry * tiy) * rinv);
    };
    cd Ea = {0.0, 0.0};
    int prev = -2;  // element whose second end point Ea belongs to
    for (int jj = j0; jj < j1; ++jj) {
        const int j = cc.start + jj;
        ScalarPtr rec = (ScalarPtr)(tab<double>(P.g, P.L.expn) + ((size_t)jside * P.N + j) * P.L.exp_stride);
        if (expanded(rec[EXP_H_CLOSE])) continue;
        const ElemRec Ej = scalar_copy(tab<ElemRec>(P.g, P.L.elem) + j);
        const double r2 = pair_r2(xi - Ej.cx, yi - Ej.cy);
        if (__builtin_amdgcn_ballot_w64(r2 < rec[LOW ? EXP_H_TAKE32 : EXP_H_TAKE64]) != 0) continue;
        cd S = {0.0, 0.0}, D = {0.0, 0.0}, Ds = {0.0, 0.0};
        for (int g = 0; g < P.q; ++g) {
            const double s = 0.5 * Ej.h * gl[g], w = 0.5 * Ej.h * gl[QMAX + g];
            const double rx = xi - fma(s, Ej.tx, Ej.cx), ry = yi - fma(s, Ej.ty, Ej.cy);
            cd h0, h1;
            const double wr = w * hankel(rx, ry, h0, h1);
            add_scaled(S, w, 1.0, h0);
            add_scaled(D, wr, fma(rx, Ej.nx, ry * Ej.ny), h1);
            if (BM) add_scaled(Ds, wr, fma(ry, tix, -rx * tiy), h1);
        }
        cd au = cmul(B.cD, D), aw = cmul(B.cS, S);
        if (BM) {
            if (prev != j - 1) Ea = end_value(Ej.ax, Ej.ay);
            const cd Eb = end_value(Ej.bx, Ej.by);
            au = cadd(au, cadd(cscale(cmul(B.cNS, S), fma(tix, Ej.tx, tiy * Ej.ty)),
                               cmul(B.cNE, {Eb.re - Ea.re, Eb.im - Ea.im})));
            aw = cadd(aw, cmul(B.cDs, Ds));
            Ea = Eb;
            prev = j;
        }
        store_entry(P.A, P.lda, P.A32, row, j, P.N, au, aw);
    }
}

// ---------------------------------------------------------------------------
// Near launch: the elements the far launch leaves, over the host's list of
// (row tile and its 64-row wave, column chunk, part of NEAR_PART elements)
// items that may hold one; one wave, one workgroup per `per` elements of an
// item.  Lanes beyond the expansion's reach take it with the general Hankel
// evaluation (series or large-argument form per lane).  The others, a few
// element lengths away or on the diagonal, go to a list in LDS and are then
// evaluated point by point, one Gauss point or end point of one pair per lane:
// with 64 consecutive rows against one element only a handful of lanes are
// that close, and a chain of q + 2 Hankel evaluations is what a small problem
// waits for.  Bound by that chain (small problems) and by FP64 VALU issue.
// Measured, Burton-Miller rows: disk of 256 elements 51 us with every element
// evaluated point by point by all lanes, 30 us with one close pair per lane,
// 15 us with one point per lane; kite of 4096 elements 296 -> 121 us.
// ---------------------------------------------------------------------------
struct NearLds {
    unsigned char todo[64 * NEAR_PART];
    double part[8][64];
};
static_assert(64 * NEAR_PART <= 256, "a list entry is one byte");

template <bool CPLX, bool BM, class T2>
__device__ __forceinline__ void near_part(const AsmArgs<T2>& P, int side, const int* __restrict__ items, int item, int per,
                                          NearLds& lds)
{
    constexpr bool LOW = sizeof(T2) == sizeof(float2);
    constexpr int NV = BM ? 8 : 4;  // partial sums of a point: S, D and, Burton-Miller rows, D*, E
    unsigned char* todo = lds.todo;
    double(*part)[64] = lds.part;
    const int parts = NEAR_PART / per;
    const int* it = items + 3 * (item / parts);
    const Tile rt = tab<Tile>(P.g, P.L.rtiles)[it[0] >> 2];
    const Tile cc = tab<Tile>(P.g, P.L.cchunks)[it[1]];
    const int j0 = it[2] * NEAR_PART + item % parts * per, cnt = min(per, cc.count - j0);
    const int lane = threadIdx.x, l0 = (it[0] & 3) * 64;
    const IfacePlan F = tab<IfacePlan>(P.g, P.L.iface)[rt.iface];
    const int d = side ? F.dr : F.dl;
    const int sg = tab<int>(P.g, P.L.sigma)[d * P.n_if + cc.iface];
    const int jside = tab<IfacePlan>(P.g, P.L.iface)[cc.iface].dr == d ? 1 : 0;
    const WaveConst W = scalar_copy(tab<WaveConst>(P.g, P.L.wave) + d);
    const BlockConst B = block_const<BM>(tab<DomConst>(P.g, P.L.dom)[d], sg);
    const ElemRec* el = tab<ElemRec>(P.g, P.L.elem);
    const int row0 = (side ? F.row_r : F.row_l) - F.off;
    const bool valid = l0 + lane < rt.count;
    const int i = rt.start + (valid ? l0 + lane : 0);
    int ntodo = 0;  // uniform
    {
        const double xi = el[i].cx, yi = el[i].cy, tix = el[i].tx, tiy = el[i].ty;
        const cd tk = {W.tkr, W.tki};
        const int cw = P.L.exp_cplx ? 2 : 1;
        const int take = P.point_launch ? (LOW ? EXP_H_TAKE32 : EXP_H_TAKE64) : LOW ? EXP_H_NEAR32 : EXP_H_NEAR64;
        for (int jj = 0; jj < cnt; ++jj) {
            const int j = cc.start + j0 + jj;
            ScalarPtr Ej = (ScalarPtr)(el + j);
            ScalarPtr rec = (ScalarPtr)(tab<double>(P.g, P.L.expn) + ((size_t)jside * P.N + j) * P.L.exp_stride);
            const double cx = Ej[E_CX], cy = Ej[E_CY], tx = Ej[E_TX], ty = Ej[E_TY];
            const double rx = xi - cx, ry = yi - cy;
            const double r2 = pair_r2(rx, ry);
            if (__builtin_amdgcn_ballot_w64(valid && r2 < rec[take]) == 0) continue;
            const bool close = valid && r2 < rec[EXP_H_CLOSE];
            const bool rest = valid && !close;
            if (__builtin_amdgcn_ballot_w64(rest) != 0) {
                auto closer = [&](double lim2) { return __builtin_amdgcn_ballot_w64(rest && r2 < lim2) != 0; };
                const int Lo = !closer(rec[EXP_H_LIM]) ? 8 : !closer(rec[EXP_H_LIM + 1]) ? 10 : !closer(rec[EXP_H_LIM + 2]) ? 12
                               : !closer(rec[EXP_H_LIM + 3]) ? 16 : 20;
                if (rest) {
                    double r, rinv;
                    sqrt_rsqrt(r2, r, rinv);
                    const double rlo = sqrt_error(rx, ry, diff_error(xi, cx, rx), diff_error(yi, cy, ry), r, rinv);
                    cd h0, h1;
                    hankel01<CPLX>(W, r, r2, rinv, rsqrt_nr(r), h0, h1, rlo);
                    const double c1 = fma(rx, tx, ry * ty) * rinv, s1 = fma(ry, tx, -rx * ty) * rinv;
                    const PairSums sums = expand<CPLX, BM, 8>(rec + EXP_HEAD, cw, Lo, h0, h1, c1, s1,
                                                              {tk.re * rinv, CPLX ? tk.im * rinv : 0.0});
                    cd au, aw;
                    combine<BM>(B, sums, fma(tix, tx, tiy * ty), fma(tiy, tx, -tix * ty), au, aw);
                    store_entry(P.A, P.lda, P.A32, (size_t)(row0 + i), j, P.N, au, aw);
                }
            }
            const unsigned long long m = __builtin_amdgcn_ballot_w64(close);
            if (close) todo[ntodo + __popcll(m & ((1ull << lane) - 1ull))] = (unsigned char)(lane * NEAR_PART + jj);
            ntodo += __popcll(m);
        }
    }
    __syncthreads();
    // close pairs: np points each (the Gauss points, then the two end points)
    const double* gl = tab<double>(P.g, P.L.gl);
    const int q = P.q, np = q + (BM ? 2 : 0), nb = 64 / np;
    const int my = lane / np, pt = lane - my * np;  // this lane's pair of the batch and point of it
    for (int t0 = 0; t0 < ntodo; t0 += nb) {
        const int nt = min(nb, ntodo - t0);
        if (my < nt) {
            const int pr = todo[t0 + my];
            const ElemRec& Ei = el[rt.start + l0 + pr / NEAR_PART];
            const ElemRec& Ej = el[cc.start + j0 + pr % NEAR_PART];
            const bool end = BM && pt >= q;
            double px, py, w = 0.0;
            if (end) {
                px = pt == q ? Ej.ax : Ej.bx;
                py = pt == q ? Ej.ay : Ej.by;
            } else {
                const double s = 0.5 * Ej.h * gl[pt];
                w = 0.5 * Ej.h * gl[QMAX + pt];
                px = Ej.cx + s * Ej.tx;
                py = Ej.cy + s * Ej.ty;
            }
            const double rx = Ei.cx - px, ry = Ei.cy - py;
            // a lane on the diagonal may sit on its own point: any distance
            // will do there, its sums are not used.  Elsewhere a point that
            // coincides has to leave a non-finite entry.
            const double d2 = fma(rx, rx, ry * ry), r2 = &Ei == &Ej ? fmax(d2, 1e-300) : d2;
            double r, rinv;
            sqrt_rsqrt(r2, r, rinv);
            cd h0, h1;
            hankel01<CPLX>(W, r, r2, rinv, rsqrt_nr(r), h0, h1);
            const double wr = w * rinv;
            const double wd = wr * fma(rx, Ej.nx, ry * Ej.ny);
            part[0][lane] = w * h0.re;
            part[1][lane] = w * h0.im;
            part[2][lane] = wd * h1.re;
            part[3][lane] = wd * h1.im;
            if constexpr (BM) {
                const double ws = wr * fma(rx, Ei.nx, ry * Ei.ny);
                part[4][lane] = ws * h1.re;
                part[5][lane] = ws * h1.im;
                const double we = end ? fma(rx, Ei.tx, ry * Ei.ty) * (pt == q ? -rinv : rinv) : 0.0;
                part[6][lane] = we * h1.re;
                part[7][lane] = we * h1.im;
            }
        }
        __syncthreads();
        if (lane < nt) {
            const int pr = todo[t0 + lane];
            const int ii = rt.start + l0 + pr / NEAR_PART, j = cc.start + j0 + pr % NEAR_PART;
            double v[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = 0.0;
            for (int g = 0; g < np; ++g)
#pragma unroll
                for (int k = 0; k < NV; ++k) v[k] += part[k][lane * np + g];
            cd sS = {v[0], v[1]}, au, aw;
            if (ii != j) {
                au = cmul(B.cD, {v[2], v[3]});
                aw = cmul(B.cS, sS);
            } else {
                // self term: D = D* = 0 on a flat element, S analytic; sS carries S / (i/4)
                const double2 sv = tab<double2>(P.g, P.L.self)[(size_t)d * P.N + ii];
                sS = cdiv({sv.x, sv.y}, B.iq);
                au = B.du;
                aw = cmul(B.cS, sS);
                if (BM) aw = cadd(aw, B.dw);
            }
            if constexpr (BM) {
                const double ninj = el[ii].nx * el[j].nx + el[ii].ny * el[j].ny;
                au = cadd(au, cadd(cscale(cmul(B.cNS, sS), ninj), cmul(B.cNE, {v[6], v[7]})));
                if (ii != j) aw = cadd(aw, cmul(B.cDs, {v[4], v[5]}));
            }
            store_entry(P.A, P.lda, P.A32, (size_t)(row0 + ii), j, P.N, au, aw);
        }
        __syncthreads();
    }
}
template <bool CPLX, bool BM, class T2>
__global__ __launch_bounds__(64, NEAR_WAVES) void k_assemble_near(const AsmArgs<T2> P, int side,
                                                                  const int* __restrict__ items, int per)
{
    __shared__ NearLds lds;
    near_part<CPLX, BM>(P, side, items, blockIdx.x, per, lds);
}

// ---------------------------------------------------------------------------
// Small systems: every variant's near and far work in one launch, the near
// work (the longer chains) first.  One wave per workgroup; a range of blocks
// belongs to one variant and kind.  CPLX: some wavenumber is complex.  Where
// one variant's work does not fill the chip, launches that follow each other
// cost more than its arithmetic, and so do the events that fork a second stream
// and join it.  bem_assemble, kite of N elements, real / lossy interior, FP64,
// us (a launch per variant and kind on two streams -> one launch): N 256  52.4
// -> 15.1 / 54.8 -> 15.8, 777  58.6 -> 41.9 / 63.4 -> 50.1, 1337  97.0 -> 80.8 /
// 111 -> 97.9, 2600  244 -> 233 / 285 -> 277, 3300  385 -> 380 / 460 -> 448,
// 4096  543 -> 566 / 647 -> 671; FP32 2600  181 -> 181 / 217 -> 217, 4096  349 ->
// 373 / 429 -> 456: the near code's registers leave three waves per SIMD to
// the far code, too, which costs most where the chip is full.
// ---------------------------------------------------------------------------
struct AsmRange {
    int end;                // first block after the range
    short kind, per;        // near 1, Burton-Miller rows 2, complex wavenumber 4, side 8; elements per wave
    int tiles;              // far: row tiles of the variant
    const int* list;        // near: items; far: row tiles
};
struct AsmRanges {
    AsmRange r[2 * ASM_VARIANTS];
};
template <bool CPLX, class T2>
__global__ __launch_bounds__(64, ALL_WAVES) void k_assemble_all(const AsmArgs<T2> P, const AsmRanges R)
{
    __shared__ NearLds lds;
    int b = blockIdx.x, k = 0, first = 0;
    while (b >= R.r[k].end) first = R.r[k++].end;
    const AsmRange r = R.r[k];
    b -= first;
    const int side = r.kind >> 3, per = r.per;
    const bool bm = r.kind & 2, cplx = CPLX && (r.kind & 4);
    if (r.kind & 1) {
        if (bm && cplx)
            near_part<CPLX, true>(P, side, r.list, b, per, lds);
        else if (cplx)
            near_part<CPLX, false>(P, side, r.list, b, per, lds);
        else if (bm)
            near_part<false, true>(P, side, r.list, b, per, lds);
        else
            near_part<false, false>(P, side, r.list, b, per, lds);
        return;
    }
    // far: the waves of a row tile, then the tiles, then the column parts
    const int li = (b % (ROW_TILE / 64)) * 64 + threadIdx.x;
    b /= ROW_TILE / 64;
    const int tile = r.list[b % r.tiles], col_part = b / r.tiles;
    if (bm && cplx)
        far_part<CPLX, true>(P, side, tile, li, col_part, per);
    else if (cplx)
        far_part<CPLX, false>(P, side, tile, li, col_part, per);
    else if (bm)
        far_part<false, true>(P, side, tile, li, col_part, per);
    else
        far_part<false, false>(P, side, tile, li, col_part, per);
}
}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_setup(char* g, const GeomLayout& L, int N, int n_dom, int q, hipStream_t s)
{
    const int eblocks = (N + SETUP_BS - 1) / SETUP_BS;
    hipLaunchKernelGGL(k_setup, dim3(1 + (3 + 2 * (EXP_LMAX + 1)) * eblocks), dim3(SETUP_BS), 0, s, g, L, N, n_dom, q, eblocks);
    return hipGetLastError();
}

namespace {

// Elements per wave: a whole chunk (far) or part (near) unless that leaves the
// chip's 1024 SIMDs short of waves; a wave's set-up costs about one element.
int elements_per_wave(int most, int least, long long waves, long long wanted)
{
    int per = most;
    while (per > least && waves * (most / per) < wanted) per /= 2;
    return per;
}

// A variant is a side of the interface, a row type and whether the wavenumber is
// complex; lists[v] / counts[v] are its row tiles, device / host.  Larger systems
// take a far and a near launch per variant, whose registers suit each; variants
// write disjoint rows, so they alternate over the two streams.
template <class T2>
hipError_t launch_variants(AsmArgs<T2> P, int n_cchunks, const int* const* lists, const int* counts,
                           const int* const* pairs, const int* pair_counts, const int* points, hipStream_t s0,
                           hipStream_t s1)
{
    const int per = elements_per_wave(COL_CHUNK, 2, (long long)((P.N + 63) / 64) * n_cchunks, 4096);
    auto launch_points = [&](int v, hipStream_t s) {
        const dim3 grid(counts[v], n_cchunks * (COL_CHUNK / per));
        const int side = v >> 2 & 1;
#define BEM_ASM_POINTS(C_, B_) \
    hipLaunchKernelGGL((k_assemble_points<C_, B_, T2>), grid, dim3(ROW_TILE), 0, s, P, side, lists[v], per)
        switch (v & 3) {
            case 0: BEM_ASM_POINTS(false, false); break;
            case 1: BEM_ASM_POINTS(true, false); break;
            case 2: BEM_ASM_POINTS(false, true); break;
            default: BEM_ASM_POINTS(true, true);
        }
#undef BEM_ASM_POINTS
    };
    if (assemble_one_launch(P.N)) {
        AsmRanges R{};
        int k = 0, end = 0;
        bool any_cplx = false;
        auto add = [&](int v, int near, int blocks, int each) {
            if (blocks == 0) return;
            end += blocks;
            const int kind = near | (v >> 1 & 1) << 1 | (v & 1) << 2 | (v >> 2 & 1) << 3;
            R.r[k++] = AsmRange{end, (short)kind, (short)each, counts[v], near ? pairs[v] : lists[v]};
            any_cplx = any_cplx || (v & 1);
        };
        for (int v = 0; v < ASM_VARIANTS; ++v) {
            const int nper = elements_per_wave(NEAR_PART, 1, pair_counts[v], 512);
            add(v, 1, pair_counts[v] * (NEAR_PART / nper), nper);
        }
        for (int v = 0; v < ASM_VARIANTS; ++v)
            add(v, 0, counts[v] * (ROW_TILE / 64) * n_cchunks * (COL_CHUNK / per), per);
        if (any_cplx)
            hipLaunchKernelGGL((k_assemble_all<true, T2>), dim3(end), dim3(64), 0, s0, P, R);
        else
            hipLaunchKernelGGL((k_assemble_all<false, T2>), dim3(end), dim3(64), 0, s0, P, R);
        for (int v = 0; v < ASM_VARIANTS; ++v)
            if (counts[v] > 0 && points[v]) launch_points(v, s0);
        return hipGetLastError();
    }
    int k = 0;
    for (int v = 0; v < ASM_VARIANTS; ++v) {
        if (counts[v] == 0) continue;
        const hipStream_t s = (k++ & 1) ? s1 : s0;
        const int bm = v >> 1 & 1, cplx = v & 1, side = v >> 2 & 1;
        const dim3 grid(counts[v], n_cchunks * (COL_CHUNK / per));
        const int nper = elements_per_wave(NEAR_PART, 1, pair_counts[v], 4096);
#define BEM_ASM_LAUNCH(C_, B_)                                                                             \
    if (cplx == C_ && bm == B_) {                                                                          \
        if (pair_counts[v] > 0)                                                                            \
            hipLaunchKernelGGL((k_assemble_near<C_, B_, T2>), dim3(pair_counts[v] * (NEAR_PART / nper)), dim3(64), 0, \
                               s, P, side, pairs[v], nper);                                                \
        hipLaunchKernelGGL((k_assemble_far<C_, B_, T2>), grid, dim3(ROW_TILE), 0, s, P, side, lists[v], per); \
    }
        BEM_ASM_LAUNCH(false, false)
        BEM_ASM_LAUNCH(true, false)
        BEM_ASM_LAUNCH(false, true)
        BEM_ASM_LAUNCH(true, true)
#undef BEM_ASM_LAUNCH
        if (points[v]) launch_points(v, s);
    }
    return hipGetLastError();
}

}  // namespace

bool assemble_one_launch(int N) { return 2 * (long long)N * N <= 1 << 24; }

hipError_t launch_assemble_f64(const char* g, const GeomLayout& L, int N, int n_if, int n_cchunks, int q,
                               const int* const* lists, const int* counts, const int* const* pairs,
                               const int* pair_counts, const int* points, bool point_launch, double2* A, size_t lda, float2* A32,
                               hipStream_t s, hipStream_t s1)
{
    return launch_variants(AsmArgs<double2>{g, L, N, n_if, q, A, A32, lda, point_launch}, n_cchunks, lists, counts, pairs,
                           pair_counts, points, s, s1);
}

hipError_t launch_assemble_f32(const char* g, const GeomLayout& L, int N, int n_if, int n_cchunks, int q,
                               const int* const* lists, const int* counts, const int* const* pairs,
                               const int* pair_counts, const int* points, bool point_launch, float2* A, size_t lda, hipStream_t s,
                               hipStream_t s1)
{
    return launch_variants(AsmArgs<float2>{g, L, N, n_if, q, A, nullptr, lda, point_launch}, n_cchunks, lists, counts, pairs,
                           pair_counts, points, s, s1);
}

}  // namespace bemk
