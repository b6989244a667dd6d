"""Rounding of the FP64 product over one group of 16 right-hand sides.

Its column splits follow the number of row blocks, down to two at n = 16384.
Whatever they are, its sums may not run longer than those of eight splits: the
rms error against extended precision, over 512 rows, is compared with that of
eight splits (sums over an eighth of the columns in both, which differ by the
order in which eight numbers are added; bound 1 % for that, where sums over half
of the columns show twice the error).
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [4096, 5999, 8192])
def test_sums_are_no_longer_than_those_of_eight_splits(N, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.kite(N, 20.0, 30.0))
    gen = torch.Generator(device="cuda").manual_seed(N)
    X = torch.view_as_complex(torch.randn(16, g.n, 2, generator=gen, device="cuda", dtype=torch.float64))
    rows = torch.linspace(0, g.n - 1, 512, device="cuda").long()
    Y = []
    for cfg in (None, "2,8,8,1"):
        if cfg:
            monkeypatch.setenv("BEM_MV_CFG", cfg)
        A = g.assemble(P.F64)  # takes the launch shapes
        Y.append(g.matvec(X)[:, rows].cpu().numpy())
    Ar = A[:, rows].cpu().numpy().astype(np.clongdouble)
    exact = X.cpu().numpy().astype(np.clongdouble) @ Ar
    err = [float(np.sqrt((np.abs(y - exact) ** 2).mean())) for y in Y]
    print(N, "rms error: built-in splits", err[0], "eight splits", err[1], flush=True)
    assert err[0] <= 1.01 * err[1]
