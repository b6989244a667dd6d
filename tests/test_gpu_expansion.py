"""The assembly's midpoint expansion at the edges of its range.

An element's Gauss sums come from one Hankel evaluation at its midpoint, with
the expansion order chosen by the element's length against the wavelength
(|k| h/2) and by its distance, and from the Gauss points one by one where no
order reaches.  Each case puts the host wavenumber just below and the interior
one just above one limit of |k| h/2, so that both choices meet in one matrix,
on meshes whose sizes straddle the 64-row waves, 32-element chunks and
4-element parts, for rules from 1 to 16 points.  All distances occur: every
element pair of a closed curve.

Reference: the oracle's entries (long double Hankel functions, point by
point).  Tolerance against the largest entry: 1e-13 as in the parity tests
(5e-13 for complex wavenumbers, whose amplitude fit is good to 2.6e-13 at
arg k = 7 degrees), plus 4 ulp of the largest phase k times the diameter, which
the oracle's own FP64 distances leave undetermined.  FP32: half an ulp of
FP32 (6e-8) and the 1e-9 of its fits and orders, doubled.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# limits of |k| h/2: order 8, 10, 12, 16, 20 of the FP64 assembly, 4, 6, 8 of
# the FP32 one, and the shortest element that is expanded
LIMITS = [1e-8, 0.026, 0.074, 0.206, 0.228, 0.495, 0.615, 1.36, 2.55]
CASES = [(lim, n, q, loss) for lim, n, q, loss in zip(
    LIMITS, [65, 128, 129, 257, 63, 97, 64, 96, 95], [8, 10, 8, 8, 16, 3, 8, 13, 8],
    [0.0, 0.0, 0.1, 0.0, 0.0, 0.1, 0.0, 0.0, 0.1])] + [(0.228, 33, 1, 0.0), (0.074, 130, 2, 0.0), (2.55, 31, 16, 0.0)]


@pytest.mark.parametrize("lim,n,q,loss", CASES, ids=[f"ka{c[0]:g}_n{c[1]}_q{c[2]}_loss{c[3]:g}" for c in CASES])
def test_entries_on_both_sides_of_an_order_limit(lim, n, q, loss):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    a = np.sin(np.pi / n)  # half an element of the inscribed n-gon
    k0, k1 = 0.999 * lim / a, 1.001 * lim / a
    spec = W.disk(n, k0, k1 * (1 + 1j * loss) if loss else k1, quad=q)
    g = P.Problem(spec)
    print("case", lim, n, q, loss, flush=True)
    Ao = O.Problem(spec).assemble()
    scale = np.abs(Ao).max()
    tol = (5e-13 if loss else 1e-13) + 4 * 2.0 ** -52 * abs(k1) * 2.0
    for prec, dt, t in ((P.F64, torch.complex128, tol), (P.F32, torch.complex64, 1.3e-7)):
        A = torch.full((g.n, g.n), complex(np.nan, np.nan), dtype=dt, device="cuda")
        g.assemble(prec, out=A)
        A = A.T.cpu().numpy().astype(np.complex128)
        assert np.isfinite(A).all()
        err = np.abs(A - Ao).max() / scale
        print(f"  {dt}: {err:.2e} (bound {t:.2e})", flush=True)
        assert err < t
