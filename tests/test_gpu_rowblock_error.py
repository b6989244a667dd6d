"""Rounding of the FP32 row-block product of few right-hand sides.

No sum may run longer than in a product of 64 column splits, formed here in
FP32 step by step from the same matrix and vectors (each fused multiply-add in
FP64, rounded; the 64 partial sums added in order): rms error over 512 rows
against FP64, bound 1.1 times (3000 errors of one size have an rms good to 2 %
each).  Sizes on both sides of 4096, where a workgroup's waves are chosen, and
the largest that takes row blocks by itself.
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _splits(Ar, X, parts=64):
    """X @ Ar in FP32, each part of the columns summed by itself."""
    n, per = Ar.shape[0], -(-Ar.shape[0] // parts)
    pad = per * parts - n
    A = np.pad(Ar, ((0, pad), (0, 0))).reshape(parts, per, -1)
    B = np.pad(X, ((0, 0), (0, pad))).reshape(len(X), parts, per)
    re = np.zeros((len(X), parts, A.shape[2]), np.float32)
    im = re.copy()
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(np.float32)
    for k in range(per):
        ar, ai = A[None, :, k].real, A[None, :, k].imag
        xr, xi = B[:, :, k, None].real, B[:, :, k, None].imag
        re = fma(-ai, xi, fma(ar, xr, re))
        im = fma(ai, xr, fma(ar, xi, im))
    s = np.zeros((len(X), A.shape[2]), np.complex64)
    for p in range(parts):
        s = (s.real + re[:, p] + 1j * (s.imag + im[:, p])).astype(np.complex64)
    return s


@pytest.mark.parametrize("N,nrhs", [(2048, 3), (2049, 3), (2400, 1), (2400, 3), (2896, 2)])
def test_sums_are_no_longer_than_those_of_64_splits(N, nrhs):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.kite(N, 20.0, 30.0))
    gen = torch.Generator(device="cuda").manual_seed(N + nrhs)
    X = torch.view_as_complex(torch.randn(nrhs, g.n, 2, generator=gen, device="cuda"))
    rows = torch.linspace(0, g.n - 1, 1536 // nrhs, device="cuda").long()
    A = g.assemble(P.F32)
    Y = g.matvec(X)[:, rows].cpu().numpy()
    Ar, Xh = A[:, rows].cpu().numpy(), X.cpu().numpy()
    exact = Xh.astype(np.complex128) @ Ar.astype(np.complex128)
    err, ref = (float(np.sqrt((np.abs(y - exact) ** 2).mean())) for y in (Y, _splits(Ar, Xh)))
    print(N, nrhs, "rms error", err, "64 splits", ref, flush=True)
    assert err <= 1.1 * ref
