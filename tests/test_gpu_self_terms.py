"""The analytic self term of elements of any length against the wavelength,
S_ii = (i / 2k) int_0^{kh/2} H0: the ascending series up to |k| h/2 = 4, steps of
a Gauss rule up to 40, the asymptotic form beyond.

Reference: mpmath's integral.  Bound 2e-14: at |k| h/2 = 4 the series' largest
term is 4 times the sum (4 ulp of it and as much again for the products), the
steps' Hankel functions are good to 2.6e-13 at most off the real axis (arg k =
5.7 degrees: 5e-14, of a part of the integral below 1/4).
"""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
mp = pytest.importorskip("mpmath")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss", [0.0, 0.1])
@pytest.mark.parametrize("ka", [1e-3, 2.0, 3.99, 4.01, 6.0, 14.0, 39.9, 40.1, 60.0])
def test_self_term(ka, loss):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    xy = W.circle_nodes(3)
    a = 0.5 * float(np.hypot(*(xy[1] - xy[0])))
    z = ka / np.hypot(1.0, loss) * (1 + 1j * loss) if loss else complex(ka)
    k0, k1 = 1.0, z / a
    g = P.Problem(W.single_material(xy, k0, k1))
    A = g.assemble(P.F64)
    got = complex(A[g.N + 0, 0])  # row 0: standard equation of the interior, column of w_0
    with mp.workdps(20):
        cuts = [0, 1e-6, 1e-4, 1e-2] + [(q + 1) / (int(ka) // 2 + 2) for q in range(int(ka) // 2 + 2)]
        I = complex(mp.quad(lambda s: mp.hankel1(0, mp.mpc(z) * s) * mp.mpc(z), sorted(set(cuts))))
    beta, eps = 1j / k0, (k1 / k0) ** 2
    want = beta * eps * (0.5j / k1) * I  # -s sigma eps S, sigma = -1
    err = abs(got - want) / abs(want)
    print(ka, loss, f"{err:.2e}", flush=True)
    assert err < 2e-14
