"""Matrices on both sides of the size up to which one launch takes all of an
assembly (2 N^2 <= 2^24: N = 2896), against rows of the oracle's.

Real and complex interiors (the single launch is compiled with and without
complex wavenumbers; both sides of the interface and both row types are in it),
FP64 and FP32; the matrix is filled with NaN first, so an entry that no range
of blocks takes shows.  Tolerance against the largest entry of a row: 1e-13
(5e-13 for complex wavenumbers, whose amplitude fit is good to 2.6e-13), plus 4
ulp of the largest phase; FP32: half an ulp (6e-8) and the 1e-9 of its fits
and orders, doubled.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss", [0.0, 0.05])
@pytest.mark.parametrize("n", [2896, 2897])
def test_rows_at_the_single_launch_limit(n, loss):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    spec = W.kite(n, 20.0, 30.0 + 1j * loss if loss else 30.0)
    g = P.Problem(spec)
    rows = np.array([0, 63, 64, 255, 256, 1500, n - 1, n, n + 1, n + 64, 2 * n - 1], dtype=np.int32)
    ref = O.Problem(spec).assemble_rows(rows)
    scale = np.abs(ref).max(axis=1, keepdims=True)
    tol = (5e-13 if loss else 1e-13) + 4 * 2.0 ** -52 * 30.0 * 3.0
    for prec, dt, t in ((P.F64, torch.complex128, tol), (P.F32, torch.complex64, 1.3e-7)):
        A = torch.full((g.n, g.n), complex(np.nan, np.nan), dtype=dt, device="cuda")
        g.assemble(prec, out=A)
        assert bool(torch.isfinite(torch.view_as_real(A)).all())
        got = A[:, torch.as_tensor(rows, device="cuda").long()].T.cpu().numpy().astype(np.complex128)
        err = (np.abs(got - ref) / scale).max()
        print(n, loss, dt, f"{err:.2e} (bound {t:.2e})", flush=True)
        assert err < t
