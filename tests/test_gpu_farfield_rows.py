"""The far field of more right-hand sides than one launch's rows of blocks hold.

Four right-hand sides to a row and 65535 rows: on both sides of 262140, and the
last one accepted (524280; one more is refused).  Every right-hand side's
pattern is that of a call of its own neighbours, bit for bit.
"""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nrhs", [262140, 262141, 262142, 524280])
def test_more_rows_than_one_launch(nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    g = P.Problem(W.single_material(W.circle_nodes(3), 1.0, 1.5))
    g.geometry()
    gen = torch.Generator(device="cuda").manual_seed(nrhs)
    X = torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda", dtype=torch.float64))
    dirs = [0.3, 1.0, 2.0, 4.0]
    F = g.farfield(X, dirs)
    for r0 in (0, 262136, nrhs - 4):
        assert torch.equal(F[r0:r0 + 4], g.farfield(X[r0:r0 + 4], dirs))
    assert torch.isfinite(torch.view_as_real(F)).all()
    if nrhs == 524280:
        with pytest.raises(P.BemError, match="too many"):
            g.farfield(torch.cat([X, X[:1]]), dirs)
