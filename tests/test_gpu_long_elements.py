"""Elements without expansion: |k| h/2 above 2.55 or below 1e-13.

Their Gauss points are evaluated one by one, by the near launch within the series
radius and half a length, beyond by the same or, where they are many, by a launch
of their own: both sides of the size up to which one launch takes the rest of an
assembly (N = 2896), few and many of them, real and
complex wavenumbers, one domain or both, rules of an odd and an even number of
points, lengths that differ along the boundary so that both kinds of element
stand beside each other in one wave.  The matrix is filled with NaN first.
Reference: rows of the oracle's; bounds against the largest entry of a row as in
the launch-limit test: 1e-13 (5e-13 complex) plus 4 ulp of the largest phase;
FP32 1.3e-7.  The near field: 1e-11 of the largest value, as at grid points.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# elements, |k0| h/2, |k1| h/2, loss, rule
CASES = [(70, 3.0, 2.4, 0.0, 8), (131, 2.4, 6.0, 0.15, 7), (300, 4.0, 5.0, 0.05, 10), (257, 0.02, 12.0, 0.1, 8),
         (65, 0.9e-13, 1.1e-13, 0.0, 8), (96, 4e-14, 5e-14, 0.1, 5), (2900, 3.0, 4.0, 0.0, 8), (2897, 0.05, 5.0, 0.1, 3),
         (600, 0.02, 2.2, 0.0, 8), (600, 2.9, 6.0, 0.05, 8), (2900, 2.2, 2.3, 0.05, 8)]


def _uneven(n):
    """A circle whose element lengths vary by a factor of 1.5."""
    t = 2 * np.pi * np.arange(n) / n
    t = t + 0.2 * np.sin(t)
    return np.stack([np.cos(t), np.sin(t)], axis=1)


@pytest.mark.parametrize("n,ka0,ka1,loss,q", CASES, ids=["-".join(f"{v:g}" for v in c) for c in CASES])
def test_rows(n, ka0, ka1, loss, q):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    a = np.pi / n
    k1 = ka1 / a
    spec = W.single_material(_uneven(n), ka0 / a, k1 * (1 + 1j * loss) if loss else k1, quad=q)
    g = P.Problem(spec)
    rows = np.unique(np.array([0, 1, 63, 64, n // 2, n - 1, n, n + 1, n + n // 2, 2 * n - 1], dtype=np.int32))
    ref = O.Problem(spec).assemble_rows(rows)
    scale = np.abs(ref).max(axis=1, keepdims=True)
    tol = (5e-13 if loss else 1e-13) + 4 * 2.0 ** -52 * max(ka0, ka1) / a * 2.0
    print("case", n, ka0, ka1, loss, q, flush=True)
    for prec, dt, t in ((P.F64, torch.complex128, tol), (P.F32, torch.complex64, 1.3e-7 + tol)):
        A = torch.full((g.n, g.n), complex(np.nan, np.nan), dtype=dt, device="cuda")
        g.assemble(prec, out=A)
        assert bool(torch.isfinite(torch.view_as_real(A)).all())
        got = A[:, torch.as_tensor(rows, device="cuda").long()].T.cpu().numpy().astype(np.complex128)
        err = (np.abs(got - ref) / scale).max()
        print(f"  {dt}: {err:.2e} (bound {t:.2e})", flush=True)
        assert err < t


@pytest.mark.parametrize("n,ka0,ka1,loss,nrhs", [(70, 3.0, 2.4, 0.0, 1), (65, 4.0, 5.0, 0.1, 3), (66, 0.1, 6.0, 0.0, 9)])
def test_field(n, ka0, ka1, loss, nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    a = np.pi / n
    k1 = ka1 / a
    spec = W.single_material(_uneven(n), ka0 / a, k1 * (1 + 1j * loss) if loss else k1, quad=16)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((2 * n, nrhs)) + 1j * rng.standard_normal((2 * n, nrhs))
    rad, th = rng.uniform(0.0, 2.0, 41), rng.uniform(0, 2 * np.pi, 41)
    rad[np.abs(rad - 1.0) < 0.3] = 0.4
    pts = np.stack([rad * np.cos(th), rad * np.sin(th)], axis=1)
    dom = (rad < 1.0).astype(np.int32)
    print("case", n, ka0, ka1, loss, nrhs, flush=True)
    Uo = O.Problem(spec).nearfield(X, pts, dom)
    g = P.Problem(spec)
    g.geometry()
    U = g.nearfield(torch.as_tensor(X.T.copy(), device="cuda"), pts, dom).cpu().numpy().T
    err = np.abs(U - Uo).max() / np.abs(Uo).max()
    print(f"  {err:.2e}", flush=True)
    assert err < 1e-11
