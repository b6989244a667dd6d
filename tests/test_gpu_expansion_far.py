"""The assembly's midpoint expansion entry by entry, away from the diagonal.

The orders' limits act on pairs beyond the close distance, whose entries are 1e-5
to 1e-2 of a matrix's largest one: here each of the four blocks (standard and
Burton-Miller rows, u and w columns) is judged by itself, a pair against the
larger of its own entry and the block's median, at wavenumbers on both sides of
a limit of |k| h/2.

Bounds, from the oracle's own rounding (its distances are FP64) with u = 2^-53:
the end-point difference is formed as E(b) - E(a), r / h <= n / pi times smaller
than its terms, 6 u n / pi; the component of a distance along a normal keeps an
absolute 4 u, against r^2 / 2 on the circle, 8 u / r^2 with r >= 3.9 h; phases
4 ulp of k times the diameter; 5e-13 for complex wavenumbers (amplitude fits off
the real axis).  FP64 entries twice all that, FP32 ones an ulp of FP32 / 2 and
1e-8, five times what the short fits and orders leave.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# |k| h/2, elements, Gauss points, loss
CASES = [(1e-8, 65, 8, 0.0), (0.026, 128, 10, 0.0), (0.074, 129, 8, 0.1), (0.206, 257, 8, 0.0), (0.228, 63, 16, 0.0),
         (0.495, 97, 3, 0.1), (0.615, 64, 8, 0.0), (1.36, 96, 13, 0.0), (2.55, 95, 8, 0.1), (0.228, 33, 1, 0.0),
         (2.55, 131, 16, 0.0)]


@pytest.mark.parametrize("lim,n,q,loss", CASES, ids=[f"ka{c[0]:g}_n{c[1]}_q{c[2]}_loss{c[3]:g}" for c in CASES])
def test_far_entries(lim, n, q, loss):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    a = np.sin(np.pi / n)
    k0, k1 = 0.999 * lim / a, 1.001 * lim / a
    spec = W.disk(n, k0, k1 * (1 + 1j * loss) if loss else k1, quad=q)
    g = P.Problem(spec)
    Ao = O.Problem(spec).assemble()
    d = np.abs((np.arange(n)[:, None] - np.arange(n)[None, :] + n // 2) % n - n // 2)
    r = 2 * np.sin(np.pi * d / n)  # of midpoints, to a factor cos(pi/n)
    far = r > 3.95 * 2 * a
    u, near = 2.0 ** -53, 3.9 * 2 * a
    tol64 = 2 * (6 * u * n / np.pi + 8 * u / near ** 2 + 8 * u * abs(k1) * 2 + (5e-13 if loss else 0))
    print("case", lim, n, q, loss, flush=True)
    worst = {}
    for prec, t in ((P.F64, tol64), (P.F32, 2.0 ** -24 + 1e-8 + tol64)):
        A = g.assemble(prec)[:, :g.n].T.cpu().numpy().astype(np.complex128)
        for rb in (0, 1):
            for cb in (0, 1):
                B, Bo = (M[rb * n:(rb + 1) * n, cb * n:(cb + 1) * n][far] for M in (A, Ao))
                e = float((np.abs(B - Bo) / np.maximum(np.abs(Bo), np.median(np.abs(Bo)))).max())
                worst[prec, rb, cb] = (e, t)
                print(f"  prec {prec} rows {rb} columns {cb}: {e:.2e} (bound {t:.2e})", flush=True)
    assert all(e < t for e, t in worst.values()), worst
