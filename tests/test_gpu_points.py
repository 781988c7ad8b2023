"""Points of small instances go through pinned memory in one launch: the same
values as by copies."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("total", [3, 40000, 65536, 65537])
def test_points(prec, total):
    """set_state and get_solution of every instance of a batch with points of
    `total` values and of others (65,536 is the longest that takes the pinned
    memory).  A point inside the bounds comes back within the two roundings of
    its scaling and, in FP32, one of its storage; with lambda the copies are
    taken, and give the same bits, for the current and the average point."""
    import paper_2508_16806_amd as pd

    m = max(1, total // 3)
    lps = [lpgen.planted(30, 70, 0.1, 1, ge_frac=0.5), lpgen.planted(m, total - m, min(1.0, 5.0 / m), 2, ge_frac=0.5),
           lpgen.planted(50, 90, 0.1, 3, ge_frac=0.5)]
    s = pd.Solver(lps, precision=prec, eps=1e-12, max_iters=64)
    rng = np.random.default_rng(0)
    pts = [(lp.l + rng.uniform(0.1, 0.9, lp.n) * (lp.u - lp.l), np.abs(rng.standard_normal(lp.m))) for lp in lps]
    for b, (x, y) in enumerate(pts):
        s.set_state(x, y, inst=b)
    rel = 2.0 ** -50 if prec == "f64" else 2.0 ** -23
    for b, want in enumerate(pts):
        for g, w in zip(s.solution(inst=b, which=pd.SOL_CURRENT), want):
            np.testing.assert_allclose(g, w, rtol=rel, atol=0)
    s.solve()
    for b in range(len(lps)):
        for which in (pd.SOL_CURRENT, pd.SOL_AVERAGE, pd.SOL_RESULT):
            x, y, _ = s.solution(inst=b, which=which, lam=True)
            for g, w in zip(s.solution(inst=b, which=which), (x, y)):
                assert np.array_equal(g, w)
