"""Small LPs (small.hip) at the edges: rows without entries beside infinite
iterates, handles of different LDS sizes side by side."""
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
