"""The tuner times the built-in shape as it times the others.

FP32, 64 right-hand sides, n = 32768: the built-in shape is within 1 % of the
best there, and its time may not be the first sample alone, taken on a GPU that
stood idle (3.9 instead of 3.5 ms, for which a slower shape was installed).
Bound 5 %.
"""
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_builtin_shape_is_timed_fairly():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2312_12787_amd as P
    P.tune_reset()
    g = P.Problem(W.kite(16384, 20.0, 30.0))
    g.assemble(P.F32)
    try:
        r = g.tune(64, reps=3)
    finally:
        P.tune_reset()
    print(r, flush=True)
    assert r["default_ms"] < 1.05 * r["best_ms"]
