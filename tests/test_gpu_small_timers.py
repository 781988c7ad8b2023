"""pdhg_time_kernels on a handle of small LPs times what its fixed steps run."""
import time

import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_sweep_times_are_the_iterations(prec):
    """An iteration by the timers against the wall clock of many in one call: the
    same within a factor of 2 (two launches an iteration would be 4 to 6 times as
    long); the handle solves as before afterwards."""
    import torch

    import paper_2508_16806_amd as pd

    lp = lpgen.planted(200, 500, 0.02, 7, ge_frac=0.5)
    s = pd.Solver(lp, precision=prec)
    assert s.sweeps() == ("small", "small")
    t = s.time_kernels(reps=50)
    assert t["ms_primal"] == t["ms_dual"] > 0
    k, best = 64 * 100, np.inf
    for _ in range(3):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        s.iterate(k)
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) * 1e3 / k)
    assert 0.5 * best <= t["ms_primal"] + t["ms_dual"] <= 2.0 * best
    s.set_state(np.zeros(lp.n), np.zeros(lp.m))
    other = pd.Solver(lp, precision=prec)
    other.set_state(np.zeros(lp.n), np.zeros(lp.m))
    assert s.solve()[0]["iters"] == other.solve()[0]["iters"]
    for a, b in zip(s.solution(), other.solution()):
        np.testing.assert_array_equal(a, b)
