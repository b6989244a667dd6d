"""Generate gauss_tables.h: the Gauss-Legendre rules of 1 to 16 points on
[-1, 1] (Sec. 7) and their even moments, rounded once from 40 digits.

Moments: GAUSS_MOM[q - 1][j] = sum_g w_g x_g^(2 j), the value the q-point rule
gives to the integral of x^(2 j) (2 / (2 j + 1) as long as 2 j < 2 q).

Run:  python gen_gauss_tables.py  (needs mpmath; writes gauss_tables.h next to it)
"""
import os

import mpmath

mpmath.mp.dps = 40

QMAX = 16
NMOM = 25


def rule(q):
    """Nodes in ascending order and weights 2 / ((1 - x^2) P_q'(x)^2)."""
    def slope(x):
        return q * (mpmath.legendre(q - 1, x) - x * mpmath.legendre(q, x)) / (1 - x * x)

    xs, ws = [], []
    for i in range(q):
        x = mpmath.cos(mpmath.pi * (i + mpmath.mpf(3) / 4) / (q + mpmath.mpf(1) / 2))
        for _ in range(8):  # Newton's method, each step doubling the digits
            x -= mpmath.legendre(q, x) / slope(x)
        if 2 * i + 1 == q:
            x = mpmath.mpf(0)
        xs.append(x)
        ws.append(2 / ((1 - x * x) * slope(x) ** 2))
    return xs[::-1], ws[::-1]


def fmt(name, rows, width):
    out = [f"static __device__ const double {name}[{len(rows)}][{width}] = {{\n"]
    for r in rows:
        out.append("    {" + ", ".join(repr(float(v)) for v in r) + "},\n")
    return "".join(out) + "};\n"


def main():
    nodes, weights, moms = [], [], []
    for q in range(1, QMAX + 1):
        x, w = rule(q)
        nodes.append(x + [0] * (QMAX - q))
        weights.append(w + [0] * (QMAX - q))
        moms.append([mpmath.fsum(b * (a ** (2 * j) if j else 1) for a, b in zip(x, w)) for j in range(NMOM)])
    out = ["/* Generated by gen_gauss_tables.py -- do not edit.\n"
           " * Gauss-Legendre rules of q = 1 .. 16 points (row q - 1, nodes ascending) and\n"
           " * their even moments sum_g w_g x_g^(2 j). */\n#pragma once\n\n",
           f"static constexpr int GAUSS_NMOM = {NMOM};\n",
           fmt("GAUSS_X", nodes, QMAX), fmt("GAUSS_W", weights, QMAX), fmt("GAUSS_MOM", moms, NMOM)]
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "gauss_tables.h")
    with open(path, "w") as f:
        f.write("".join(out))
    print("wrote", path)


if __name__ == "__main__":
    main()
