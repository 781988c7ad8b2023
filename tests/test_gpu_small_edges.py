"""Small LPs (small.hip) at the edges: rows without entries beside infinite
iterates, handles of different LDS sizes side by side, no rows, periods longer
than a launch."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_empty_rows_ignore_the_others(prec):
    """A row or column without entries does not see its neighbours, also where
    their iterates are infinite: bit for bit the step it takes beside finite ones."""
    import paper_2508_16806_amd as pd

    rng = np.random.default_rng(4)
    m, n = 90, 250
    A = np.where(rng.random((m, n)) < 0.04, 1.0, 0.0)
    rows, cols = np.arange(5, m, 7), np.arange(3, n, 5)
    A[rows] = 0.0
    A[:, cols] = 0.0
    lp = lpgen.from_dense(A, rng.integers(0, 2, m), rng.standard_normal(m), rng.standard_normal(n),
                          np.full(n, -np.inf), np.full(n, np.inf))
    got = []
    for big in (0.0, np.inf):
        s = pd.Solver(lp, precision=prec, ruiz_iters=0, step_size=0.1, primal_weight=1.0)
        x, y = np.linspace(-1, 1, n), np.linspace(0, 1, m)
        x[np.setdiff1d(np.arange(n), cols)] = big
        y[np.setdiff1d(np.arange(m), rows)] = big
        s.set_state(x, y)
        s.iterate(3)
        x, y = s.solution(which=pd.SOL_CURRENT)
        assert big == 0.0 or not np.isfinite(x).all()
        got.append((x[cols], y[rows]))
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_a_smaller_handle_beside_a_larger_one(prec):
    """A handle whose LP fills most of the LDS launches as before after one with
    a tiny LP was set up, with and without recorded launches (graphs)."""
    import paper_2508_16806_amd as pd

    lp = lpgen.planted(1003, 2501, 0.005, 6, ge_frac=0.5)
    for graph in (0, 1):
        kw = dict(precision=prec, max_iters=128, use_graph=graph, unroll_capacity=8, unroll_checkpoint=2)
        a = pd.Solver(lp, **kw)
        a.solve()
        want = a.solution()
        a = pd.Solver(lp, **kw)
        b = pd.Solver(lpgen.tiny(3, n=5, m=3), **kw)
        b.solve()
        a.solve()
        for u, v in zip(a.solution(), want):
            np.testing.assert_array_equal(u, v)
        a.iterate(8, record=True)
        assert np.isfinite(a.backward(np.ones(lp.n), np.ones(lp.m))["c"]).all()


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_no_rows(prec):
    """Without rows k steps take x from x0 to clip(x0 - k tau c): the rounding of
    each step, at most 4 of the storage's units of 1 + |x|."""
    import paper_2508_16806_amd as pd

    n, k = 70, 9
    c = np.linspace(-1.0, 1.0, n)
    lp = lpgen.from_dense(np.zeros((0, n)), [], [], c, np.zeros(n), np.full(n, 2.0))
    s = pd.Solver(lp, precision=prec, ruiz_iters=0, step_size=0.1, primal_weight=1.0)
    assert s.sweeps() == ("small", "small")
    s.set_state(np.ones(n), np.zeros(0))
    s.iterate(k)
    x, y = s.solution(which=pd.SOL_CURRENT)
    unit = 2.0 ** (-24 if prec == "f32" else -53)
    np.testing.assert_allclose(x, np.clip(1.0 - k * s.info()["tau"] * c, 0.0, 2.0), rtol=0, atol=4 * k * unit * 3.0)
    assert y.size == 0


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("every", [255, 256, 257, 600])
def test_periods_longer_than_a_launch(prec, every):
    """Check periods around and beyond the 256 steps of a launch, with averages and
    restarts: the iterates, average and counts of the tiled sweeps, bit for bit."""
    import paper_2508_16806_amd as pd

    lp, big = lpgen.planted(300, 700, 0.02, 4, ge_frac=0.5), lpgen.planted(2000, 5000, 0.006, 9)
    kw = dict(precision=prec, check_every=every, max_iters=4 * every, eps=1e-14)
    a, b = pd.Solver(lp, **kw), pd.Solver([lp, big], batch_resident_bytes=0, **kw)
    assert a.sweeps() == ("small", "small") and b.sweeps(0) == ("direct", "direct")
    ra, rb = a.solve()[0], b.solve()[0]
    assert (ra["iters"], ra["restarts"], ra["kkt"]) == (rb["iters"], rb["restarts"], rb["kkt"])
    assert ra["restarts"] > 0
    for which in (pd.SOL_CURRENT, pd.SOL_AVERAGE):
        for u, v in zip(a.solution(which=which), b.solution(which=which)):
            np.testing.assert_array_equal(u, v)
