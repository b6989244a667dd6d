"""Generate hankel_tables.h: polynomial fits of the Hankel amplitude functions
used by the device Hankel evaluator for |z| >= XS.

For nu = 0, 1 write H_nu^(1)(z) = sqrt(2/(pi z)) e^{i(z - nu pi/2 - pi/4)} P_nu(z).
On the real axis P_nu(x) = M_nu(x) + i N_nu(x) with M, N real-analytic, smooth
and non-oscillatory; their asymptotic expansions are even (M) and odd (N) in
1/x.  With w = (XS/x)^2 in [0, 1] and u = XS/x we fit
    M_nu(x) ~ m_nu(w),   N_nu(x) ~ u n_nu(w)
by Chebyshev interpolation in w (mpmath at high precision as ground truth,
converted to monomials in w in high precision and rounded once).  The same
polynomials, evaluated at complex w, continue analytically to complex z with
small argument (lossy media).

Run:  python gen_hankel_tables.py  (needs mpmath; writes hankel_tables.h next to it)
"""
import os

import mpmath

mpmath.mp.dps = 60

XS64 = 6.0      # FP64 path: series below, fit above
DEG64 = 14
# Below XS64 the four entire functions of t = (z/2)^2: ascending series about t = 0
# for |z| < ZLOW, Taylor series about TMID beyond (to |z| = 6 the ascending series
# would add terms 60 times its sum), NMID terms for the range of real z, NWIDE for
# that of lossy wavenumbers (to |z| = 7)
ZLOW = 3.0
NLOW = 15
TMID = 5.5
NMID = 16
NWIDE = 19
XS32 = 4.0      # FP32 path
DEG32 = 6


def amplitude(nu, x):
    x = mpmath.mpf(x)
    return mpmath.hankel1(nu, x) / (mpmath.sqrt(2 / (mpmath.pi * x))
                                    * mpmath.exp(1j * (x - nu * mpmath.pi / 2 - mpmath.pi / 4)))


def fit(nu, xs, deg):
    K = deg + 1
    nodes = [(mpmath.cos(mpmath.pi * (k + mpmath.mpf(1) / 2) / K) + 1) / 2 for k in range(K)]  # w in (0,1)
    mvals, nvals = [], []
    for w in nodes:
        x = xs / mpmath.sqrt(w)
        P = amplitude(nu, x)
        mvals.append(mpmath.re(P))
        nvals.append(mpmath.im(P) * x / xs)
    # Chebyshev interpolation coefficients in t = 2w - 1
    def cheb_coeffs(vals):
        c = []
        for j in range(K):
            s = mpmath.mpf(0)
            for k in range(K):
                s += vals[k] * mpmath.cos(mpmath.pi * j * (k + mpmath.mpf(1) / 2) / K)
            c.append(2 * s / K)
        c[0] /= 2
        return c

    def to_monomial_w(c):
        # sum c_j T_j(2w - 1) -> sum a_m w^m
        n = len(c)
        T_prev = [mpmath.mpf(1)] + [mpmath.mpf(0)] * (n - 1)        # T_0
        T_cur = [mpmath.mpf(-1), mpmath.mpf(2)] + [mpmath.mpf(0)] * (n - 2)  # T_1 = 2w - 1
        a = [c[0] * v for v in T_prev]
        if n > 1:
            a = [a[i] + c[1] * T_cur[i] for i in range(n)]
        for j in range(2, n):
            # T_{j} = 2 (2w - 1) T_{j-1} - T_{j-2}
            T_next = [mpmath.mpf(0)] * n
            for i in range(n):
                T_next[i] -= 2 * T_cur[i] + T_prev[i]
                if i + 1 < n:
                    T_next[i + 1] += 4 * T_cur[i]
            a = [a[i] + c[j] * T_next[i] for i in range(n)]
            T_prev, T_cur = T_cur, T_next
        return a

    return to_monomial_w(cheb_coeffs(mvals)), to_monomial_w(cheb_coeffs(nvals))


def check(nu, xs, mco, nco, dtype_eps):
    worst = 0.0
    for j in range(400):
        x = xs * (1 + 0.01 * j) if j < 200 else xs * 3 * (200.0 / xs) ** ((j - 200) / 199.0)
        w = (xs / x) ** 2
        m = 0.0
        for a in reversed(mco):
            m = m * w + float(a)
        n = 0.0
        for a in reversed(nco):
            n = n * w + float(a)
        P = complex(m, n * xs / x)
        ref = complex(amplitude(nu, x))
        worst = max(worst, abs(P - ref) / abs(ref))
    return worst


def fmt(name, coeffs, ctype):
    suffix = "f" if ctype == "float" else ""
    body = ",\n    ".join(repr(float(c)) + suffix for c in coeffs)
    return f"static constexpr {ctype} {name}[{len(coeffs)}] = {{\n    {body}}};\n"


def series_constants(nterms):
    """Coefficients in t = (z/2)^2 of the ascending series (DLMF 10.2.2, 10.8.1, 10.8.2):
    J0 = sum j0_m t^m,  Y0 = (2/pi)(ln(z/2) + gamma) J0 + sum e0_m t^m,
    J1 = (z/2) sum j1_m t^m,  Y1 = -(2/pi)/z + (2/pi) ln(z/2) J1 + (z/2) sum e1_m t^m."""
    j0, e0, j1, e1 = [], [], [], []
    H = mpmath.mpf(0)
    for m in range(nterms):
        if m > 0:
            H += mpmath.mpf(1) / m
        sgn = (-1) ** m
        f = mpmath.factorial(m)
        f1 = mpmath.factorial(m + 1)
        j0.append(mpmath.mpf(sgn) / (f * f))
        e0.append(mpmath.mpf(0) if m == 0 else (2 / mpmath.pi) * (-sgn) * H / (f * f))
        j1.append(mpmath.mpf(sgn) / (f * f1))
        psi = mpmath.digamma(m + 1) + mpmath.digamma(m + 2)
        e1.append(-(1 / mpmath.pi) * psi * sgn / (f * f1))
    return j0, e0, j1, e1


def about(c, t0, nterms):
    """The first coefficients in t - t0 of sum_m c_m t^m."""
    return [mpmath.fsum(c[m] * mpmath.binomial(m, k) * mpmath.mpf(t0) ** (m - k) for m in range(k, len(c)))
            for k in range(nterms)]


def main():
    out = ['/* Generated by gen_hankel_tables.py -- do not edit.\n'
           ' * Monomial coefficients (ascending powers of w = (XS/z)^2) of the fitted\n'
           ' * Hankel amplitude functions: P_nu(z) = m_nu(w) + i (XS/z) n_nu(w),\n'
           ' * H_nu^(1)(z) = sqrt(2/(pi z)) e^{i(z - nu pi/2 - pi/4)} P_nu(z), |z| >= XS. */\n',
           '#pragma once\n\n']
    for tag, xs, deg in [("F64", XS64, DEG64), ("F32", XS32, DEG32)]:
        out.append(f"static constexpr double HANKEL_XS_{tag} = {xs!r};\n")
        out.append(f"static constexpr int HANKEL_NC_{tag} = {deg + 1};\n")
        for nu in (0, 1):
            mco, nco = fit(nu, xs, deg)
            err = check(nu, xs, mco, nco, 0)
            out.append(f"/* nu = {nu}: max relative amplitude error on the real axis (double Horner) {err:.2e} */\n")
            ctype = "double" if tag == "F64" else "float"
            out.append(fmt(f"HANKEL_M{nu}_{tag}", mco, ctype))
            out.append(fmt(f"HANKEL_N{nu}_{tag}", nco, ctype))
            print(tag, nu, f"{err:.2e}")
    out.append("/* J0, Y0 = (2/pi)(ln(z/2) + gamma) J0 + E0, J1 = (z/2) J1', Y1 = -(2/pi)/z + (2/pi) ln(z/2) J1 + (z/2) E1\n"
               " * (DLMF 10.2.2, 10.8.1, 10.8.2); J0, E0, J1', E1 as series in t = (z/2)^2 for |z| < SERIES_ZLOW,\n"
               " * in t - SERIES_TMID up to |z| = HANKEL_XS_F64 (SERIES_NMID terms) or 7 (SERIES_NWIDE). */\n")
    out.append(f"static constexpr double SERIES_ZLOW = {ZLOW!r}, SERIES_TMID = {TMID!r};\n")
    out.append(f"static constexpr int SERIES_NLOW = {NLOW}, SERIES_NMID = {NMID}, SERIES_NWIDE = {NWIDE};\n")
    for name, c in zip(("J0", "E0", "J1", "E1"), series_constants(60)):
        out.append(fmt(f"LOW_{name}", c[:NLOW], "double"))
        out.append(fmt(f"MID_{name}", about(c, TMID, NWIDE), "double"))
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "hankel_tables.h")
    with open(path, "w") as f:
        f.write("".join(out))
    print("wrote", path)


if __name__ == "__main__":
    main()
