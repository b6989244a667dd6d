"""The far-field kernel at the edges of its blocks, against the oracle.

A block takes two directions of one right-hand side, or three directions of
four; a launch up to 384 directions; its 256 threads the elements.  The coarse
polygon's elements are long against the wavelength (both forms of sin(a)/a);
the one moved far from the origin has phases beyond 2^29, which take the
library's reduction.  Bound: 1e-13 of the largest value, plus 4 ulp of the
largest phase k0 |c|, which both sides round before taking its sine.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# elements, k0, right-hand sides, directions, shift
CASES = [(8, 5.0, 1, 1, 0.0), (3, 1.0, 2, 2, 0.0), (255, 3.0, 4, 7, 0.0), (256, 20.0, 5, 384, 0.0),
         (257, 50.0, 9, 385, 0.0), (600, 30.0, 1, 383, 0.0), (64, 2.0, 3, 5, 4e8)]


@pytest.mark.parametrize("n,k0,nrhs,ndir,shift", CASES, ids=["-".join(f"{v:g}" for v in c) for c in CASES])
def test_farfield_matches_the_oracle(n, k0, nrhs, ndir, shift):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    spec = W.single_material(W.circle_nodes(n, center=(shift, 0.0)), k0, 1.5 * k0)
    rng = np.random.default_rng(n)
    X = rng.standard_normal((2 * n, nrhs)) + 1j * rng.standard_normal((2 * n, nrhs))
    dirs = rng.uniform(0, 2 * np.pi, ndir)
    g = P.Problem(spec)
    g.geometry()
    F = g.farfield(torch.as_tensor(X.T.copy(), device="cuda"), dirs).cpu().numpy().T
    Fo = O.Problem(spec).farfield(X, dirs)
    err = np.abs(F - Fo).max() / np.abs(Fo).max()
    tol = 1e-13 + 4 * 2.0 ** -52 * k0 * (shift + 1.0)
    print(n, nrhs, ndir, f"error {err:.2e} bound {tol:.2e}", flush=True)
    assert err < tol
