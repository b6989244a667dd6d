// nearfield.hip -- the field at points off the boundary (Sec. 7.1: the total
// field at field points), from the boundary data of a solution.
//
// A point x of domain d takes the representation formula of that domain:
//   u(x) = [d = host] u_in(x) + sum_m sigma_dm sum_{j in m} (eps_d S_j(x) w_j - D_j(x) u_j),
//   S_j(x) = int_j G_d(x - y) ds_y,  D_j(x) = int_j dG_d/dn_y(x - y) ds_y,
// sigma_dm = +1 where the normal of interface m leaves domain d.
// Element integrals: the element's q-point Gauss rule when x is at least two
// element lengths away (Bernstein-ellipse error below 1e-14); closer, the
// Laplace parts of the kernels, -(1/2pi) ln r and (1/2pi) (x-y).n / r^2, and
// the next log terms, (k^2/8pi) r^2 ln r of the single layer and
// -(k^2/4pi) (x-y).n ln r of the double layer, are integrated in closed form
// over the straight element and Gauss is applied to what remains of
// (i/4) H0(kr) and (ik/4) H1(kr) (x-y).n / r, on each side of the foot of the
// perpendicular from x.
//
// A point beyond an element's close distance takes its Gauss rule from one
// Hankel evaluation at the midpoint (expansion_dev.h; that distance is about
// four element lengths, so the rule applies there by the first line); one
// without expansion (|k| h/2 outside EXP_KA_MIN .. EXP_KA_MAX) point by point
// beyond 5/2 lengths from the midpoint (1024 elements at |k| h/2 = 4, 101 x 101
// points: 0.84 ms; 5.14 ms as close pairs).
//
// Layout: points xy[2 p], xy[2 p + 1], domain dom[p]; X column-major [u; w]
// per right-hand side (ldx); U column-major, point fastest (ldu).
//  * k_nearfield, one launch per domain (uniform wavenumber and Hankel
//    constants): all pairs beyond the close distance, and the incident field.
//    A wave takes a few points x several elements at a time (64 points would
//    leave most of the chip idle on the paper's 101 x 101 grid, 64 elements
//    would read 64 records at every load); the sums of a workgroup's waves are
//    added in a fixed order.
//  * k_nearfield_close, one launch: a wave looks over a few points, lanes over
//    the elements; where a point has close elements they are evaluated and
//    added to its value.
// Bound by FP64 VALU issue.  Measured, 101 x 101 points, 1024 elements: 805 us
// with every Gauss point evaluated and one wave per point; now 229 us (2 x 100 us
// and, the close pairs, 41 us, which took 94 us with one pair per lane).
#include <hip/hip_runtime.h>

#include "expansion_dev.h"
#include "hankel_dev.h"
#include "internal.h"
#include "launch.h"

namespace bemk {

namespace {

constexpr int NF_BS = 256;
constexpr double INV_2PI = 0.15915494309189533577;

template <class T>
__device__ __forceinline__ const T* tab(const char* g, size_t off) { return reinterpret_cast<const T*>(g + off); }

// int_{u0}^{u1} ln sqrt(u^2 + xn^2) du
__device__ __forceinline__ double log_integral(double u0, double u1, double xn)
{
    auto F = [&](double u) {
        const double r2 = fma(u, u, xn * xn);
        double v = (u != 0.0 ? u * 0.5 * log(r2) : 0.0) - u;
        if (xn != 0.0) v += xn * atan(u / xn);
        return v;
    };
    return F(u1) - F(u0);
}

// int_{u0}^{u1} (u^2 + xn^2) ln sqrt(u^2 + xn^2) du
__device__ __forceinline__ double r2log_integral(double u0, double u1, double xn)
{
    const double d2 = xn * xn;
    auto F = [&](double u) {
        const double r2 = fma(u, u, d2);
        const double u3 = u * u * u;
        double v = (u != 0.0 ? (u3 / 6.0 + d2 * u * 0.5) * log(r2) : 0.0) - u3 / 9.0 + d2 * u / 3.0 - d2 * u;
        if (xn != 0.0) v += (d2 * xn - d2 * xn / 3.0) * atan(u / xn);
        return v;
    };
    return F(u1) - F(u0);
}

// What the integrals of one close pair have in closed form, and the segment
// data of its Gauss points: beyond two lengths (far) one segment, the whole
// element, and nothing in closed form; else the element on each side of the
// foot of the perpendicular from x, and the log terms.
struct CloseGeom {
    double xt, xn, cut;  // x along the element from node a, (x - y).n, the foot
    bool far;
    __device__ __forceinline__ CloseGeom(const ElemRec& E, double x, double y)
    {
        const double dx = x - E.ax, dy = y - E.ay;
        xt = dx * E.tx + dy * E.ty;
        xn = dx * E.nx + dy * E.ny;  // for every y on the element
        const double h = E.h;
        const double ut = xt < 0.0 ? -xt : (xt > h ? xt - h : 0.0);
        far = sqrt(fma(ut, ut, xn * xn)) >= 2.0 * h;
        cut = fmin(fmax(xt, 0.0), h);
    }
};

// Gauss point g of one part (0, 1) of a close pair: its contributions to S and
// D (for a far pair without the factors i/4 and i k/4).
template <bool CPLX>
__device__ __forceinline__ void close_term(const WaveConst& W, cd k, const ElemRec& E, const CloseGeom& C, int part,
                                           double xg, double wt, double x, double y, cd& S, cd& D)
{
    S = {0.0, 0.0};
    D = {0.0, 0.0};
    const double h = E.h;
    double half, rx = 0.0, ry = 0.0, r2;
    if (C.far) {
        if (part == 1) return;
        half = 0.5 * h;
        const double sg = half * xg;
        rx = x - (E.cx + sg * E.tx);
        ry = y - (E.cy + sg * E.ty);
        r2 = fma(rx, rx, ry * ry);
    } else {
        const double s0 = part == 0 ? 0.0 : C.cut, s1 = part == 0 ? C.cut : h;
        half = 0.5 * (s1 - s0);
        if (half <= 0.0) return;
        const double u = C.xt - fma(half, xg, 0.5 * (s0 + s1));  // (x - y).t
        r2 = fma(u, u, C.xn * C.xn);
    }
    double r, rinv;
    sqrt_rsqrt(r2, r, rinv);
    cd h0, h1;
    hankel01<CPLX>(W, r, r2, rinv, rsqrt_nr(r), h0, h1);
    const double wg = half * wt;
    if (C.far) {
        S = {wg * h0.re, wg * h0.im};
        const double wd = wg * (rx * E.nx + ry * E.ny) * rinv;
        D = {wd * h1.re, wd * h1.im};
        return;
    }
    const cd ik4 = {-0.25 * k.im, 0.25 * k.re};
    const cd k2 = cmul(k, k);
    const cd c4 = cscale(k2, 0.5 * INV_2PI * C.xn);  // (k^2 / 4 pi) xn
    const cd c8 = cscale(k2, 0.25 * INV_2PI);        // k^2 / 8 pi
    // (i/4) H0 + (1/2pi) ln r - (k^2 / 8 pi) r^2 ln r
    const double lnr = log(r);
    const double lr2 = wg * r2 * lnr;
    S.re = fma(wg, -0.25 * h0.im + INV_2PI * lnr, -lr2 * c8.re);
    S.im = fma(wg, 0.25 * h0.re, -lr2 * c8.im);
    // [(ik/4) H1 - 1/(2 pi r)] xn / r + (k^2 / 4 pi) xn ln r
    const cd q = cmul(ik4, h1);
    const double f = wg * C.xn * rinv;
    const double lr = wg * lnr;
    D.re = fma(f, q.re - INV_2PI * rinv, lr * c4.re);
    D.im = fma(f, q.im, lr * c4.im);
}

// S and D of a close pair from the sums of its terms: the closed forms of the
// Laplace parts, of the double layer's log term
//   (ik/4) H1(kr) xn / r = xn / (2 pi r^2) - (k^2 / 4 pi) xn ln r + smooth
// and of the single layer's
//   (1/2pi) ln r (1 - J0(kr)) = (k^2 / 8 pi) r^2 ln r + O(r^4 ln r).
__device__ __forceinline__ void close_sums(cd k, const ElemRec& E, const CloseGeom& C, cd sr, cd dr, cd& S, cd& D)
{
    if (C.far) {  // S = (i/4) sum w H0, D = (ik/4) sum w H1 (r.n)
        S = {-0.25 * sr.im, 0.25 * sr.re};
        D = cmul({-0.25 * k.im, 0.25 * k.re}, dr);
        return;
    }
    const double h = E.h, xt = C.xt, xn = C.xn;
    const double lnint = log_integral(-xt, h - xt, xn);
    const cd k2 = cmul(k, k);
    const cd DLog = cscale(k2, -0.5 * INV_2PI * xn * lnint);
    const cd SLog = cscale(k2, 0.25 * INV_2PI * r2log_integral(-xt, h - xt, xn));
    S = {sr.re - INV_2PI * lnint + SLog.re, sr.im + SLog.im};
    D = {dr.re + INV_2PI * atan2(xn * h, fma(xn, xn, -xt * (h - xt))) + DLog.re, dr.im + DLog.im};
}

// orders the wave's LDS writes before its later reads (the other waves of the
// workgroup are elsewhere)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// sum over the wave's 64 lanes in a fixed butterfly order (every lane ends
// with the same value)
__device__ __forceinline__ double wave_add(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Workgroup of k_nearfield: 4 points, 4 waves, so that a wave's 4 points x 16
// elements step seldom mixes the two Hankel forms and the waves fill the chip
// (paper's grid: 8 waves 286, 8 points 293, 2 points 262, 4 points 252 us).
constexpr int NF_PTS = 4, NF_WAVES = 4, NF_EL = 64 / NF_PTS;
constexpr int NFC_PTS = 4;  // points a wave of k_nearfield_close looks over

// Squared distance of a point and an element's midpoint, the same in both
// kernels: each pair is taken by one of them.
__device__ __forceinline__ double midpoint_r2(double x, double y, const ElemRec& E)
{
    const double rx = x - E.cx, ry = y - E.cy;
    return fma(rx, rx, ry * ry);
}

// the record of element j in domain d, one of the two sides of interface P
__device__ __forceinline__ const double* exp_record(const char* g, const GeomLayout& L, int N, const IfacePlan& P, int d,
                                                    int j)
{
    return tab<double>(g, L.expn) + ((size_t)(P.dr == d ? 1 : 0) * N + j) * L.exp_stride;
}

// The sums S and Gn of an element without expansion, point by point; (rx, ry)
// from its midpoint.
template <bool CPLX>
__device__ __forceinline__ PairSums rule_sums(const WaveConst& W, const ElemRec& E, const double* __restrict__ gl, int nq,
                                              double rx, double ry)
{
    PairSums Q;
    Q.S = Q.Gn = {0.0, 0.0};
    const double half = 0.5 * E.h;
    for (int i = 0; i < nq; ++i) {
        const double s = half * gl[i], w = half * gl[QMAX + i];
        const double px = fma(-s, E.tx, rx), py = fma(-s, E.ty, ry), r2 = fma(px, px, py * py);
        double r, rinv;
        sqrt_rsqrt(r2, r, rinv);
        cd h0, h1;
        hankel01<CPLX>(W, r, r2, rinv, rsqrt_nr(r), h0, h1);
        add_scaled(Q.S, w, 1.0, h0);
        add_scaled(Q.Gn, w * rinv, fma(px, E.nx, py * E.ny), h1);
    }
    return Q;
}

// POINTS: the domain has elements without expansion.
template <bool CPLX, int RB, bool POINTS>
__global__ __launch_bounds__(64 * NF_WAVES, RB > 4 ? 2 : 3) void k_nearfield(const char* __restrict__ g, GeomLayout L, int n_if,
                                                                 int N, int nq, int d, const double2* __restrict__ X,
                                                                 size_t ldx, int nr, NearAngles ang, int add_incident,
                                                                 const double* __restrict__ xy,
                                                                 const int* __restrict__ dom, int npts,
                                                                 double2* __restrict__ U, size_t ldu)
{
    __shared__ double2 sums[NF_WAVES][RB][NF_PTS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int pl = lane & (NF_PTS - 1), ph = lane / NF_PTS;
    const int p = blockIdx.x * NF_PTS + pl;
    const bool act = p < npts && dom[min(p, npts - 1)] == d;
    if (__builtin_amdgcn_ballot_w64(act) == 0) return;  // the same points in every wave
    const double x = xy[2 * (size_t)min(p, npts - 1)], y = xy[2 * (size_t)min(p, npts - 1) + 1];
    const WaveConst W = tab<WaveConst>(g, L.wave)[d];
    const DomConst Dm = tab<DomConst>(g, L.dom)[d];
    const cd k = {Dm.k[0], Dm.k[1]};
    const cd eps = {Dm.eps[0], Dm.eps[1]};
    const ElemRec* el = tab<ElemRec>(g, L.elem);
    const int cw = L.exp_cplx ? 2 : 1;
    cd acc[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) acc[r] = {0.0, 0.0};
    for (int m = 0; m < n_if; ++m) {
        const int sg = tab<int>(g, L.sigma)[d * n_if + m];
        if (sg == 0) continue;
        const IfacePlan P = tab<IfacePlan>(g, L.iface)[m];
        // eps sigma S = cS sum w H0, sigma D = cD sum w H1 (r.n)/r
        const cd cS = cscale(cmul(eps, {0.0, 0.25}), (double)sg);
        const cd cD = cscale({-0.25 * k.im, 0.25 * k.re}, (double)sg);
        for (int e0 = wave * NF_EL; e0 < P.count; e0 += NF_WAVES * NF_EL) {
            const int j = P.off + min(e0 + ph, P.count - 1);
            const double* rec = exp_record(g, L, N, P, d, j);
            const double cx = el[j].cx, cy = el[j].cy, tx = el[j].tx, ty = el[j].ty;
            const double rx = x - cx, ry = y - cy;
            const double r2 = midpoint_r2(x, y, el[j]);
            const bool on = act && e0 + ph < P.count && !(r2 < el[j].close2[P.dr == d]);
            if (__builtin_amdgcn_ballot_w64(on) == 0) continue;
            auto closer = [&](double lim2) { return __builtin_amdgcn_ballot_w64(on && r2 < lim2) != 0; };
            const int Lo = !closer(rec[EXP_H_LIM]) ? 8 : !closer(rec[EXP_H_LIM + 1]) ? 10 : !closer(rec[EXP_H_LIM + 2]) ? 12
                           : !closer(rec[EXP_H_LIM + 3]) ? 16 : 20;
            if (on) {
                PairSums Q;
                if (!POINTS || rec[EXP_H_CLOSE] < __longlong_as_double(0x7ff0000000000000ll)) {
                    double r, rinv;
                    sqrt_rsqrt(r2, r, rinv);
                    const double rlo = sqrt_error(rx, ry, diff_error(x, cx, rx), diff_error(y, cy, ry), r, rinv);
                    cd h0, h1;
                    hankel01<CPLX>(W, r, r2, rinv, rsqrt_nr(r), h0, h1, rlo);
                    Q = expand<CPLX, false, 8>(rec + EXP_HEAD, cw, Lo, h0, h1, fma(rx, tx, ry * ty) * rinv,
                                               fma(ry, tx, -rx * ty) * rinv,
                                               {W.tkr * rinv, CPLX ? W.tki * rinv : 0.0});
                } else {
                    Q = rule_sums<CPLX>(W, el[j], tab<double>(g, L.gl), nq, rx, ry);
                }
                const cd eS = cmul(cS, Q.S), sD = cmul(cD, Q.Gn);
#pragma unroll
                for (int q = 0; q < RB; ++q) {
                    if (q < nr) {
                        const double2 u = X[(size_t)q * ldx + j], w = X[(size_t)q * ldx + N + j];
                        acc[q].re += eS.re * w.x - eS.im * w.y - (sD.re * u.x - sD.im * u.y);
                        acc[q].im += eS.re * w.y + eS.im * w.x - (sD.re * u.y + sD.im * u.x);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
        cd v = acc[r];  // the elements of a step, then the waves in turn
#pragma unroll
        for (int o = NF_PTS; o < 64; o *= 2) {
            v.re += __shfl_xor(v.re, o, 64);
            v.im += __shfl_xor(v.im, o, 64);
        }
        if (ph == 0) sums[wave][r][pl] = make_double2(v.re, v.im);
    }
    __syncthreads();
    if (wave != 0 || !act) return;
    for (int r = ph; r < nr; r += NF_EL) {
        cd v = {0.0, 0.0};
        for (int w = 0; w < NF_WAVES; ++w) {
            v.re += sums[w][r][pl].x;
            v.im += sums[w][r][pl].y;
        }
        if (d == 0 && add_incident) {
            double sn, cs;
            sincos(ang.v[r], &sn, &cs);
            double ps, pc;
            sincos(k.re * (cs * x + sn * y), &ps, &pc);
            v.re += pc;
            v.im += ps;
        }
        U[(size_t)r * ldu + p] = make_double2(v.re, v.im);
    }
}

// Adds the close pairs of point p to its value; one wave.  The close elements
// are listed in LDS (up to 64 at a time), their Gauss points evaluated one per
// lane -- a point has about seven close elements, and one lane per pair would
// be a chain of 2 q evaluations -- and each pair finished by one lane.
struct CloseScratch {
    int list[64];
    double part[4][64];
};
template <bool CPLX>
__device__ __forceinline__ void close_point(const char* __restrict__ g, const GeomLayout& L, int n_if, int N, int q,
                                            const double2* __restrict__ X, size_t ldx, int nr,
                                            const double* __restrict__ xy, int p, int d, double2* __restrict__ U,
                                            size_t ldu, CloseScratch& sc)
{
    const double x = xy[2 * (size_t)p], y = xy[2 * (size_t)p + 1];
    const ElemRec* el = tab<ElemRec>(g, L.elem);
    const int lane = threadIdx.x & 63;
    const WaveConst W = tab<WaveConst>(g, L.wave)[d];
    const DomConst Dm = tab<DomConst>(g, L.dom)[d];
    const cd k = {Dm.k[0], Dm.k[1]};
    const double* gl = tab<double>(g, L.gl);
    const int np = 2 * q, nb = 64 / np;  // terms of a pair, pairs of a batch
    const int my = lane / np, part = (lane - my * np) / q, gi = lane - my * np - part * q;
    cd acc[NF_RB];
#pragma unroll
    for (int r = 0; r < NF_RB; ++r) acc[r] = {0.0, 0.0};
    int n = 0;  // listed pairs (uniform)
    auto flush = [&](int sg) {
        cd sr = {0.0, 0.0}, dr = {0.0, 0.0};
        for (int t0 = 0; t0 < n; t0 += nb) {
            wave_sync();
            if (my < nb && t0 + my < n) {
                const ElemRec& E = el[sc.list[t0 + my]];
                cd S, D;
                close_term<CPLX>(W, k, E, CloseGeom(E, x, y), part, gl[gi], gl[QMAX + gi], x, y, S, D);
                sc.part[0][lane] = S.re;
                sc.part[1][lane] = S.im;
                sc.part[2][lane] = D.re;
                sc.part[3][lane] = D.im;
            }
            wave_sync();
            if (lane >= t0 && lane < min(n, t0 + nb))
                for (int t = 0; t < np; ++t) {
                    const int a = (lane - t0) * np + t;
                    sr.re += sc.part[0][a];
                    sr.im += sc.part[1][a];
                    dr.re += sc.part[2][a];
                    dr.im += sc.part[3][a];
                }
        }
        if (lane < n) {
            const int j = sc.list[lane];
            cd S, D;
            close_sums(k, el[j], CloseGeom(el[j], x, y), sr, dr, S, D);
            const cd eS = cscale(cmul({Dm.eps[0], Dm.eps[1]}, S), (double)sg);
            const cd sD = cscale(D, (double)sg);
#pragma unroll
            for (int r = 0; r < NF_RB; ++r) {
                if (r < nr) {
                    const double2 u = X[(size_t)r * ldx + j], w = X[(size_t)r * ldx + N + j];
                    acc[r].re += eS.re * w.x - eS.im * w.y - (sD.re * u.x - sD.im * u.y);
                    acc[r].im += eS.re * w.y + eS.im * w.x - (sD.re * u.y + sD.im * u.x);
                }
            }
        }
        wave_sync();
        n = 0;
    };
    for (int m = 0; m < n_if; ++m) {
        const int sg = tab<int>(g, L.sigma)[d * n_if + m];
        if (sg == 0) continue;
        const IfacePlan P = tab<IfacePlan>(g, L.iface)[m];
        for (int e0 = 0; e0 < P.count; e0 += 64) {
            const int j = P.off + min(e0 + lane, P.count - 1);
            const bool on = e0 + lane < P.count && midpoint_r2(x, y, el[j]) < el[j].close2[P.dr == d];
            const unsigned long long mask = __builtin_amdgcn_ballot_w64(on);
            const int more = __popcll(mask);
            if (more == 0) continue;
            if (n + more > 64) flush(sg);
            if (on) sc.list[n + __popcll(mask & ((1ull << lane) - 1ull))] = j;
            n += more;
        }
        if (n) flush(sg);
    }
#pragma unroll
    for (int r = 0; r < NF_RB; ++r) {
        if (r >= nr) continue;
        const cd v = {wave_add(acc[r].re), wave_add(acc[r].im)};
        if (lane == 0) {
            const double2 u = U[(size_t)r * ldu + p];
            U[(size_t)r * ldu + p] = make_double2(u.x + v.re, u.y + v.im);
        }
    }
}

// CPLX: some wavenumber is complex.  A workgroup looks over NFC_PTS points per
// wave for close elements, then its waves take the points that have some in
// turn (neighbours on a grid often have some together).
template <bool CPLX>
__global__ __launch_bounds__(NF_BS, 2) void k_nearfield_close(const char* __restrict__ g, GeomLayout L, int n_if,
                                                              int N, int q, const double2* __restrict__ X,
                                                              size_t ldx, int nr, const double* __restrict__ xy,
                                                              const int* __restrict__ dom, int npts,
                                                              double2* __restrict__ U, size_t ldu)
{
    constexpr int NW = NF_BS / 64;
    __shared__ CloseScratch sc[NW];
    __shared__ unsigned hits[NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int b0 = blockIdx.x * NW * NFC_PTS, p0 = b0 + wave * NFC_PTS;
    const ElemRec* el = tab<ElemRec>(g, L.elem);
    double px[NFC_PTS], py[NFC_PTS];
    int pd[NFC_PTS];
#pragma unroll
    for (int a = 0; a < NFC_PTS; ++a) {
        const int p = min(p0 + a, npts - 1);
        px[a] = xy[2 * (size_t)p];
        py[a] = xy[2 * (size_t)p + 1];
        pd[a] = p0 + a < npts ? dom[p] : -1;
    }
    unsigned hit = 0;
    for (int m = 0; m < n_if; ++m) {
        const IfacePlan P = tab<IfacePlan>(g, L.iface)[m];
#pragma unroll 4
        for (int e = lane; e < P.count; e += 64) {
            const ElemRec& E = el[P.off + e];
#pragma unroll
            for (int a = 0; a < NFC_PTS; ++a) {
                const double lim = pd[a] == P.dr ? E.close2[1] : pd[a] == P.dl ? E.close2[0] : 0.0;
                hit |= midpoint_r2(px[a], py[a], E) < lim ? 1u << a : 0u;
            }
        }
    }
    unsigned any = 0;
#pragma unroll
    for (int a = 0; a < NFC_PTS; ++a)
        if (__builtin_amdgcn_ballot_w64((hit >> a & 1u) != 0) != 0) any |= 1u << a;
    if (lane == 0) hits[wave] = any;
    __syncthreads();
    int turn = 0;
    for (int w = 0; w < NW; ++w)
        for (unsigned m = __builtin_amdgcn_readfirstlane(hits[w]); m != 0; m &= m - 1) {
            if (turn++ % NW != wave) continue;
            const int p = b0 + w * NFC_PTS + __builtin_ctz(m);
            close_point<CPLX>(g, L, n_if, N, q, X, ldx, nr, xy, p, __builtin_amdgcn_readfirstlane(dom[p]), U, ldu,
                              sc[wave]);
        }
}

}  // namespace

hipError_t launch_nearfield(const char* g, const GeomLayout& L, int n_if, int n_dom, int N, int q, const int* dom_cplx,
                            const int* dom_points, const double2* X, size_t ldx, int nrhs, const double* angles,
                            const double* xy, const int* dom, int npts, double2* U, size_t ldu, hipStream_t s)
{
    bool cplx = false;
    for (int d = 0; d < n_dom; ++d) cplx = cplx || dom_cplx[d];
    for (int r0 = 0; r0 < nrhs; r0 += NF_RB) {
        const int nr = nrhs - r0 < NF_RB ? nrhs - r0 : NF_RB;
        NearAngles ang{};
        for (int r = 0; r < nr; ++r) ang.v[r] = angles ? angles[r0 + r] : 0.0;
        const double2* Xr = X + (size_t)r0 * ldx;
        double2* Ur = U + (size_t)r0 * ldu;
        const int inc = angles ? 1 : 0;
        for (int d = 0; d < n_dom; ++d) {
#define BEM_NF_LAUNCH(C_, R_, P_)                                                                                       \
    hipLaunchKernelGGL((k_nearfield<C_, R_, P_>), dim3((npts + NF_PTS - 1) / NF_PTS), dim3(64 * NF_WAVES), 0, s, g, L, n_if, \
                       N, q, d, Xr, ldx, nr, ang, inc, xy, dom, npts, Ur, ldu)
            if (dom_cplx[d] && dom_points[d])
                BEM_NF_LAUNCH(true, NF_RB, true);
            else if (dom_points[d])
                BEM_NF_LAUNCH(false, NF_RB, true);
            else if (dom_cplx[d]) {
                if (nr == 1)
                    BEM_NF_LAUNCH(true, 1, false);
                else
                    BEM_NF_LAUNCH(true, NF_RB, false);
            } else {
                if (nr == 1)
                    BEM_NF_LAUNCH(false, 1, false);
                else if (nr <= 4)
                    BEM_NF_LAUNCH(false, 4, false);
                else
                    BEM_NF_LAUNCH(false, NF_RB, false);
            }
#undef BEM_NF_LAUNCH
        }
        const int per = NFC_PTS * (NF_BS / 64);  // points per workgroup
        const dim3 grid((npts + per - 1) / per);
        if (cplx)
            hipLaunchKernelGGL(k_nearfield_close<true>, grid, dim3(NF_BS), 0, s, g, L, n_if, N, q, Xr, ldx, nr,
                               xy, dom, npts, Ur, ldu);
        else
            hipLaunchKernelGGL(k_nearfield_close<false>, grid, dim3(NF_BS), 0, s, g, L, n_if, N, q, Xr, ldx, nr,
                               xy, dom, npts, Ur, ldu);
    }
    return hipGetLastError();
}

}  // namespace bemk
