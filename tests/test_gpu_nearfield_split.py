"""The near field where its two kernels meet: pairs beyond the close distance
(one Hankel evaluation at the element's midpoint) and close pairs (Gauss
points and closed forms), at the edges of their groupings.

Points from one to more than a workgroup's worth, one to nine right-hand sides
(the kernels for 1, up to 4 and up to 8, and a second group), rules of 8, 10
and 16 points (4, 3 and 2 close pairs per batch), and a mesh so coarse that
every element is a close one (|k| h/2 above the expansion's limit, 130
elements: the list of 64 fills more than once).  Reference: the oracle's
adaptive integrals; bounds as in the near-field parity test for the same
quantities: 1e-11 of the largest value at grid points, 1e-9 within 0.3 element
lengths of the boundary.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# name, elements, k0, k1, rule, right-hand sides, points
CASES = [("one_point", 70, 5.0, 7.0, 8, 1, 1), ("tail", 64, 5.0, 7.0, 10, 3, 21), ("lossy", 90, 6.0, 8.0 + 0.4j, 8, 2, 40),
         ("two_groups", 65, 3.0, 4.0, 8, 9, 35), ("all_close", 130, 110.0, 120.0, 16, 4, 37)]


@pytest.mark.parametrize("name,n,k0,k1,q,nrhs,npts", CASES, ids=[c[0] for c in CASES])
def test_both_kernels_against_the_oracle(name, n, k0, k1, q, nrhs, npts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    spec = W.disk(n, k0, k1, quad=q)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((2 * n, nrhs)) + 1j * rng.standard_normal((2 * n, nrhs))
    # alternately anywhere within radius 2 and 1e-4 .. 0.3 lengths off the polygon
    h, r_in = 2 * np.sin(np.pi / n), np.cos(np.pi / n)
    th = 2 * np.pi * (rng.integers(0, n, npts) + 0.5) / n
    off = h * 10.0 ** rng.uniform(-4, np.log10(0.3), npts) * rng.choice([-1.0, 1.0], npts)
    close = np.arange(npts) % 2 == 1
    rad = np.where(close, r_in + off, rng.uniform(0.0, 2.0, npts))
    rad[~close & (np.abs(rad - 1.0) < 2 * h)] = 0.5
    pts = np.stack([rad * np.cos(th), rad * np.sin(th)], axis=1)
    dom = (rad < r_in).astype(np.int32)
    ang = rng.uniform(0, 2 * np.pi, nrhs)
    print("case", name, flush=True)
    Uo = O.Problem(spec).nearfield(X, pts, dom, angles=ang)
    g = P.Problem(spec)
    g.geometry()
    Xd = torch.as_tensor(X.T.copy(), device="cuda")
    U = g.nearfield(Xd, pts, dom, angles=ang).cpu().numpy().T
    err = np.abs(U - Uo).max(axis=1) / np.abs(Uo).max()
    print(f"  grid {err[~close].max():.2e}  close {err[close].max() if close.any() else 0:.2e}", flush=True)
    assert err[~close].max() < 1e-11 and (not close.any() or err[close].max() < 1e-9)
    # a point that is no number gives none, in either domain
    bad = g.nearfield(Xd, np.array([[np.nan, 0.0], [0.1, np.nan]]), np.array([0, 1], dtype=np.int32), angles=ang)
    assert torch.isnan(torch.view_as_real(bad)).any(dim=-1).all()
