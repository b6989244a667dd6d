"""Rounding of the Hankel functions where the series would cancel (|k r| 2 to 6; to 7
where Im k > 0.07 Re k, the amplitude fits being good to 1e-13 there at |k r| = 6).

With a one-point rule an entry of a standard row's single-layer block is the
element's length times H0 at the distance of two midpoints.  A polygon of 128
elements puts all pairs' |k r| between 0 and 5.95 (8).  Reference: mpmath.  The rms
of the relative errors within each unit of |k r|, bound 6e-16 = twice what
follows from H0 itself (2.5e-16) and five more roundings (length, moment, factor,
two products: 0.6e-16 each); complex k: twice the bound, for as many products
again and sums of opposite signs; four times it at arg k = 5.7 degrees (the fits
are good to 1e-15 at |k r| = 7).
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
mp = pytest.importorskip("mpmath")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss,top", [(0.0, 2.975), (0.02, 2.975), (0.1, 4.0)])
def test_single_layer_entries(loss, top):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    n, k0, k1 = 128, 1.0, top / abs(1 + 1j * loss) * (1 + 1j * loss) if loss else top
    xy = W.circle_nodes(n) * np.array([1.0, 0.93])
    g = P.Problem(W.single_material(xy, k0, k1, quad=1))
    A = g.assemble(P.F64)[:, :g.n].T.cpu().numpy()
    c = 0.5 * (xy + np.roll(xy, -1, axis=0))
    rng = np.random.default_rng(0)
    i, j = rng.integers(0, n, 3000), rng.integers(0, n, 3000)
    i, j = i[i != j], j[i != j]
    err, kr = [], []
    with mp.workdps(30):
        k = mp.mpc(complex(k1))
        f = mp.mpc(0, 1) / k0 * (k / k0) ** 2 * mp.mpc(0, 0.25)  # beta eps i/4
        for a, b in zip(i, j):
            r = mp.hypot(mp.mpf(c[a, 0]) - mp.mpf(c[b, 0]), mp.mpf(c[a, 1]) - mp.mpf(c[b, 1]))
            e = (b + 1) % n
            h = mp.hypot(mp.mpf(xy[e, 0]) - mp.mpf(xy[b, 0]), mp.mpf(xy[e, 1]) - mp.mpf(xy[b, 1]))
            want = f * h * mp.hankel1(0, k * r)
            err.append(float(abs(mp.mpc(complex(A[a, n + b])) - want) / abs(want)))
            kr.append(float(abs(k) * r))
    err, kr = np.array(err), np.array(kr)
    worst = 0.0
    for u in range(int(np.ceil(2 * top))):
        m = (kr >= u) & (kr < u + 1)
        rms = float(np.sqrt((err[m] ** 2).mean()))
        print(u, int(m.sum()), f"{rms:.2e} max {err[m].max():.2e}", flush=True)
        worst = max(worst, rms)
    assert worst < (6e-16 if not loss else 1.2e-15 if loss < 0.05 else 2.4e-15)
