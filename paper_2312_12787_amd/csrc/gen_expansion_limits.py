"""The limits of the midpoint expansions' orders (EXP_X*, EXP_KA*, EXP32_* of
internal.h; expansion_dev.h has the expansions).

An element of half length a at distance r, x = a / r, ka = |k| a.  Order L drops
the Hankel orders above L.  Criterion: the dropped part of every sum, over r and
the angle phi, relative to that sum's scale,
    S: mu_0 |H_0|,   Gt, Gn: mu_0 |H_1|,   Tt, Tn: nu_1 max(|H_0|, |H_2|),
stays below a target, 4e-17 (FP64) or 1e-9 (FP32), for real k, once for large r
(the limit of ka) and once over r at ka below that (the limit of x).  The
constants are the limits found here, less 2 to 5 %.

What the limits leave is then measured the strict way: the magnitudes of the
dropped terms added up, without the signs of H_p and of cos p phi, against the
largest magnitude among the orders 0 to 2 of the same sum; for real k and at
arg k = 10 degrees, the most lossy one.

Run:  python gen_expansion_limits.py  (needs mpmath; prints, writes nothing)
"""
import mpmath

mpmath.mp.dps = 40

# order, x, ka as in internal.h
FP64 = [(8, 0.0087, 0.074), (10, 0.0223, 0.228), (12, 0.0415, 0.495), (16, 0.0855, 1.36), (20, 0.128, 2.55)]
FP32 = [(4, 0.0054, 0.026), (6, 0.0306, 0.206), (8, 0.0725, 0.615), (16, 0.2, 2.55)]
ANGLES = [mpmath.mpf(p) for p in (0, 0.3, 0.8, 1.2)] + [mpmath.pi / 2]
SUMS = ("S", "Gt", "Gn", "Tt", "Tn")


def rule(q):
    """Gauss-Legendre nodes and weights."""
    xs, ws = [], []
    for i in range(q):
        x = mpmath.cos(mpmath.pi * (i + mpmath.mpf(3) / 4) / (q + mpmath.mpf(1) / 2))
        for _ in range(8):
            d = q * (mpmath.legendre(q - 1, x) - x * mpmath.legendre(q, x)) / (1 - x * x)
            x -= mpmath.legendre(q, x) / d
        xs.append(x)
        ws.append(2 / ((1 - x * x) * d * d))
    return xs, ws


RULE = rule(8)


def coefficients(ka, top):
    """Per sum the factors of H_p (times cos or sin of p phi), a = 1."""
    xs, ws = RULE
    mu = [mpmath.fsum(w * mpmath.besselj(m, ka * x) for x, w in zip(xs, ws)) for m in range(top + 2)]
    nu = [2 * mpmath.besselj(m, ka) for m in range(top + 2)]
    c = {s: [mpmath.mpf(0)] * (top + 1) for s in SUMS}
    for p in range(top + 1):
        if p % 2 == 0:
            c["S"][p] = mu[p] * (2 if p else 1)
            c["Tt"][p] = nu[p - 1] - nu[p + 1] if p else -nu[1]
            c["Tn"][p] = nu[p - 1] + nu[p + 1] if p else mpmath.mpf(0)
        else:
            c["Gt"][p] = mu[p - 1] - mu[p + 1]
            c["Gn"][p] = mu[p - 1] + mu[p + 1]
    return c


def hankels(z, top):
    H = [mpmath.hankel1(0, z), mpmath.hankel1(1, z)]
    for p in range(1, top):
        H.append(2 * p / z * H[p] - H[p - 1])
    return H


def dropped(L, ka, z):
    """The criterion: largest dropped part over the sums and angles."""
    top = L + 10
    c, H = coefficients(ka, top), hankels(z, top)
    mu0, nu1 = c["S"][0], -c["Tt"][0]
    scale = {"S": mu0 * abs(H[0]), "Gt": mu0 * abs(H[1]), "Tt": nu1 * max(abs(H[0]), abs(H[2]))}
    scale["Gn"], scale["Tn"] = scale["Gt"], scale["Tt"]
    worst = mpmath.mpf(0)
    for s in SUMS:
        f = mpmath.sin if s in ("Gn", "Tn") else mpmath.cos
        for phi in ANGLES:
            worst = max(worst, abs(mpmath.fsum(c[s][p] * H[p] * f(p * phi) for p in range(L + 1, top + 1))) / scale[s])
    return worst


def largest(ok, lo, hi, steps=18):
    for _ in range(steps):
        m = mpmath.sqrt(lo * hi)
        lo, hi = (m, hi) if ok(m) else (lo, m)
    return lo


def left(L, x, ka, arg):
    """Strict measure at the limit: {sum: largest over r}."""
    top = L + 14
    k = ka * mpmath.expj(arg)
    c = coefficients(k, top)
    out = {s: mpmath.mpf(0) for s in SUMS}
    for z in [k / x * f for f in (1, 1.3, 2, 4, 10)]:
        H = hankels(z, top)
        for s in SUMS:
            t = [abs(c[s][p] * H[p]) for p in range(top + 1)]
            out[s] = max(out[s], mpmath.fsum(t[L + 1:]) / max(t[:3]))
    return out


def main():
    for name, table, target in (("FP64", FP64, mpmath.mpf("4e-17")), ("FP32", FP32, mpmath.mpf("1e-9"))):
        for L, x, ka in table:
            if L < 16 or name == "FP64":  # FP32's order 16 is chosen for its reach, far below the target
                kl = largest(lambda k: max(dropped(L, k, mpmath.mpf(z)) for z in (L, 2 * L, 4 * L, 200)
                                           if z > 1.2 * k) < target, mpmath.mpf("1e-4"), mpmath.mpf(6))
                xl = min(largest(lambda v: dropped(L, k, k / v) < target, mpmath.mpf("1e-5"), mpmath.mpf("0.6"))
                         for k in (f * kl for f in (1e-4, 0.1, 0.5, 1)))
                print(f"{name} order {L}: found ka {float(kl):.4g}, x {float(xl):.4g}; used {ka}, {x}", flush=True)
        for arg in (0, 10):
            worst = {s: mpmath.mpf(0) for s in SUMS}
            for L, x, ka in table:
                for f in (1e-3, 0.3, 1):
                    r = left(L, mpmath.mpf(x), f * mpmath.mpf(ka), mpmath.radians(arg))
                    worst = {s: max(worst[s], r[s]) for s in SUMS}
            print(f"{name}, arg k = {arg} degrees:", "  ".join(f"{s} {float(worst[s]):.1e}" for s in SUMS), flush=True)


if __name__ == "__main__":
    main()
