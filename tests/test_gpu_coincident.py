"""A collocation point on another element's quadrature or end point.

The sums of such a pair do not exist (H0 and H1 at distance zero).  Two squares
that touch along an edge meshed differently on its two sides, so that a node of
one is the midpoint of an element of the other, or meshed alike with a rule
that has a point at the midpoint: the matrix has to show it in a non-finite
entry and the solve has to refuse it; only an element against itself, whose
entry is analytic, may pass over its own midpoint.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _squares(shift, quad):
    """[0, 2]^2 with unit elements and [2, 4] x [shift, shift + 2]."""
    a = W.square_nodes(2, 2.0) + 1.0
    b = W.square_nodes(2, 2.0) + np.array([3.0, 1.0 + shift])
    spec = W.single_material(a, 1.3, 2.1, quad=quad)
    spec.k.append(1.7 + 0j)
    spec.interfaces.append(W.Interface(b, True, 2, 0))
    return spec


@pytest.mark.parametrize("shift,quad", [(0.5, 8), (0.0, 3), (0.0, 1)])
@pytest.mark.parametrize("prec", ["F64", "F32", "MIXED"])
def test_coincident_points_are_refused(shift, quad, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    g = P.Problem(_squares(shift, quad))
    A = g.assemble(getattr(P, prec))
    assert not torch.isfinite(torch.view_as_real(A[:, :g.n])).all()
    with pytest.raises(P.BemError, match="NONFINITE"):
        g.solve(g.rhs([0.3]), restart=20, tol=1e-8)


@pytest.mark.parametrize("quad", [1, 3, 8])
def test_apart_they_pass(quad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    spec = _squares(0.0, quad)
    spec.interfaces[1].xy = spec.interfaces[1].xy + np.array([0.25, 0.0])
    g = P.Problem(spec)
    assert torch.isfinite(torch.view_as_real(g.assemble(P.F64)[:, :g.n])).all()
