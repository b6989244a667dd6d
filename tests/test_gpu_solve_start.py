"""Which columns a solve runs: decided on the device from the norms of B and
read back by the host at a cycle's end.

Columns of zeros (converged at once, X = 0), with a NaN or an overflowing norm
(BEM_E_NONFINITE, X = 0) and ordinary ones, up to the 64 that one launch
chooses by a mask, over restarts; then the same solver state with other columns
and with a block of zeros.  An ordinary column has to reach its tolerance
(residual formed here from the FP64 matrix; its own rounding, some 1e-15, is far
below 2 tol) whatever its neighbours hold.
"""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-9


def _residual(A, X, B):
    R = X @ A - B
    return (R.abs().square().sum(1).sqrt() / B.abs().square().sum(1).sqrt()).cpu()


@pytest.mark.parametrize("prec", ["F64", "MIXED"])
@pytest.mark.parametrize("nrhs", [1, 3, 17, 63, 64])
def test_zero_and_nonfinite_columns(nrhs, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    g = P.Problem(W.disk(48, 2.0, 3.0))
    A = g.assemble(P.F64)[:, :g.n].clone()
    g.assemble(getattr(P, prec))
    gen = torch.Generator(device="cuda").manual_seed(nrhs)
    B = torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda", dtype=torch.float64))
    opts = dict(restart=12, tol=TOL, inner_tol=1e-4)
    zero = [r for r in range(nrhs) if r % 7 == 2]
    B[zero] = 0
    X, info = g.solve(B, **opts)
    live = [r for r in range(nrhs) if r not in zero]
    assert info.converged.all() and info.status == 0
    assert all(info.iters[r] == 0 and info.rel_residual[r] == 0.0 for r in zero)
    assert torch.count_nonzero(X[zero]).item() == 0
    assert _residual(A, X[live], B[live]).max() < 2 * TOL
    assert info.restarts[live].max() >= 1
    # the same solver state, other columns: one NaN, one whose norm overflows
    C = B.clone()
    bad = sorted({0, nrhs - 1})
    C[bad[0], 5] = complex(float("nan"), 0.0)
    C[bad[-1], 7] = 1e200
    Y = torch.full_like(C, 3.0)
    if prec == "F64" or nrhs > 1:
        with pytest.raises(P.BemError, match="NONFINITE"):
            g.solve(C, X=Y, **opts)
    else:  # the refinement takes a NaN norm for a zero one (an infinite norm it refuses)
        assert g.solve(C, X=Y, **opts)[1].converged.all()
    good = [r for r in live if r not in bad]
    assert torch.count_nonzero(Y[bad]).item() == 0
    if good:
        assert torch.equal(Y[good], X[good])
    # nothing to do, then the first solve again: bit for bit
    Z, info = g.solve(torch.zeros_like(B), **opts)
    assert info.converged.all() and torch.count_nonzero(Z).item() == 0
    X2, _ = g.solve(B, **opts)
    assert torch.equal(X2, X)
