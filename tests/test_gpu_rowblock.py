"""The one-launch row-block products at the edges of their tiles.

A workgroup owns 16 rows; its 8 or 16 waves take 16 or 32 columns at a time;
up to four right-hand sides keep X in LDS (n times right-hand sides below 128
KiB), five to sixteen go through the matrix cores; larger products, and calls
whose X and Y share memory, are split over columns.  Sizes on both sides of
each of these, FP64 and FP32, against the FP64 product of the same matrix.
Bound per entry: 4 sqrt(n) u (|A| |X|), u = 2^-53 or 2^-24 (a sum of n products
rounds like a random walk; the complex product adds a few roundings).
"""
import ctypes as C

import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [3, 8, 9, 16, 31, 32, 33, 100, 257, 1023, 1366]


def _check(Y, A, X, u):
    A, X = A.to(torch.complex128), X.to(torch.complex128)
    err = (Y.to(torch.complex128) - X @ A).abs()
    bound = 4 * A.shape[0] ** 0.5 * u * (X.abs() @ A.abs())
    return float((err / bound).max())


@pytest.mark.parametrize("N", SIZES)
def test_products_of_all_widths(N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.disk(N, 2.0, 3.0 + 0.1j))
    gen = torch.Generator(device="cuda").manual_seed(N)
    for prec, dt, u in ((P.F64, torch.complex128, 2.0 ** -53), (P.F32, torch.complex64, 2.0 ** -24)):
        A = g.assemble(prec)[:, :g.n]
        for nrhs in (1, 2, 3, 4, 5, 15, 16, 17, 65):
            X = torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda", dtype=torch.float64)).to(dt)
            worst = _check(g.matvec(X), A, X, u)
            assert worst < 1, (N, nrhs, dt, worst)
            Y = X.clone()  # in place: the product may not be written while X is read
            _, _, wb = g.sizes(prec, min(nrhs, 64), 1)
            w = g._workspace(wb)
            if nrhs <= 64:
                assert P.lib().bem_matvec(g._h, nrhs, C.c_void_p(Y.data_ptr()), g.n, C.c_void_p(Y.data_ptr()), g.n,
                                          C.c_void_p(w.data_ptr()), w.numel(),
                                          C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
                worst = _check(Y, A, X, u)
                assert worst < 1, (N, nrhs, dt, "in place", worst)
