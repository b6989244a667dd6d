"""Products through the matrix cores with split columns: splits by the number of
row blocks (128 or 64 rows each) and of blocks that run at once.

Sizes just above the row-block limits of 16 right-hand sides (FP64 n 4096, FP32
5792), a full turn of 64 row blocks and the one beyond it, two turns; with more
right-hand sides also both sides of n = 3072, below which a wave takes one row
tile, and tiny systems; ragged last row block and last split.  Against the FP64 product of the same matrix; bound per entry: 4 sqrt(n)
u (|A| |X|), u = 2^-53 or 2^-24 (a sum of n products rounds like a random walk;
the complex product adds a few roundings).
"""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [20, 77, 1535, 1536, 2049, 2753, 2901, 4096, 4097, 5999])
def test_products_split_by_row_blocks(N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.disk(N, 2.0, 3.0 + 0.1j))
    gen = torch.Generator(device="cuda").manual_seed(N)
    for prec, dt, u in ((P.F64, torch.complex128, 2.0 ** -53), (P.F32, torch.complex64, 2.0 ** -24)):
        A = g.assemble(prec)[:, :g.n]
        wide = A.to(torch.complex128)
        size = A.abs().double()
        for nrhs in (5, 16, 17, 33, 64):
            X = torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda", dtype=torch.float64)).to(dt)
            err = (g.matvec(X).to(torch.complex128) - X.to(torch.complex128) @ wide).abs()
            bound = 4 * g.n ** 0.5 * u * (X.abs().double() @ size)
            worst = float((err / bound).max())
            assert worst < 1, (N, nrhs, dt, worst)


def test_wide_products_fit_the_scratch_they_fitted():
    """64 right-hand sides at n = 2674, 11 splits: 31.3 of the 32 MiB that a
    product without a workspace may take (12 splits would be refused)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.disk(1337, 2.0, 3.0 + 0.1j))
    g.assemble(P.F64)
    X = torch.randn(64, g.n, 2, device="cuda", dtype=torch.float64, generator=torch.Generator(device="cuda").manual_seed(1))
    X = torch.view_as_complex(X)
    assert torch.equal(g.matvec_noalloc(X), g.matvec(X))
