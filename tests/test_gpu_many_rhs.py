"""Solves with more right-hand sides than one pass over the matrix takes (64).

They run as blocks of 64, so each block's solution is that of a call with its
columns alone, bit for bit; a column without convergence or a non-finite one in
any block gives the whole call's status.
"""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _problem(P, n, prec, nrhs, seed):
    g = P.Problem(W.disk(n, 2.0, 3.0 + 0.1j))
    g.assemble(prec)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return g, torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda", dtype=torch.float64))


@pytest.mark.parametrize("prec", ["F64", "MIXED"])
@pytest.mark.parametrize("nrhs,graph", [(65, 0), (64 + 17, 3), (128, 0), (200, 0)])
def test_blocks_of_64(nrhs, graph, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    g, B = _problem(P, 48, getattr(P, prec), nrhs, nrhs)
    opts = dict(restart=30, tol=1e-9, inner_tol=1e-4, graph_steps=graph)
    X, info = g.solve(B, **opts)
    assert info.status == 0 and info.converged.all() and len(info.iters) == nrhs
    for r0 in range(0, nrhs, 64):
        Xb, ib = g.solve(B[r0:r0 + 64], **opts)
        assert torch.equal(X[r0:r0 + 64], Xb)
        assert (info.iters[r0:r0 + 64] == ib.iters).all()
    # one column of the last block does not converge, then is no number
    assert g.solve(B, **{**opts, "max_iter": 2, "max_refine": 1})[1].status == 6
    C = B.clone()
    C[70 if nrhs > 70 else 64, 3] = 1e200
    with pytest.raises(P.BemError, match="NONFINITE"):
        g.solve(C, **opts)


def test_batch_of_unequal_counts():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    items = [_problem(P, n, P.F64, nrhs, n) for n, nrhs in ((48, 70), (33, 3), (64, 130))]
    opts = dict(restart=30, tol=1e-9)
    for (g, B), (X, info) in zip(items, P.solve_batch([g for g, _ in items], [B for _, B in items], **opts)):
        Xa, ia = g.solve(B, **opts)
        assert info.converged.all() and torch.equal(X, Xa) and (info.iters == ia.iters).all()


def test_served_request_of_more_than_64():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    from paper_2312_12787_amd import serve as S
    spec, angles = W.disk(64, 2.0, 3.0), W.equispaced_angles(70)
    with S.Server(1 << 30, slots=2, prec=P.MIXED, dirs=W.equispaced_angles(36)) as srv:
        ids = [srv.submit(spec, a) for a in (angles, angles[:64], angles[64:])]
        res = {r.id: r for r in srv.drain()}
    whole, first, rest = (res[i] for i in ids)
    assert all(r.status == 0 for r in res.values()) and whole.nrhs == 70
    assert (whole.far_field[:64] == first.far_field).all() and (whole.far_field[64:] == rest.far_field).all()
