"""The sweeps in two passes (spread.hip): the row-binned sweeps to the bit."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _lp(m, n, nnz, longest, seed, transpose):
    """Rows of 0 to 2,000 entries and one of `longest` over random columns."""
    import scipy.sparse as sp

    rng = np.random.default_rng(seed)
    lens = np.minimum(rng.zipf(1.6, m), 2000) - 1
    lens = np.minimum(lens * max(1, nnz // max(1, lens.sum())), 2000)
    lens[m // 2] = longest
    rows = np.repeat(np.arange(m), lens)
    K = sp.csr_matrix((rng.uniform(0.5, 1.5, rows.size), (rows, rng.integers(0, n, rows.size))), shape=(m, n))
    K.sum_duplicates()
    if transpose:
        K = K.T.tocsr()
    K.sort_indices()
    m, n = K.shape
    x = rng.uniform(0, 1, n)
    return lpgen.LP(n, m, K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data,
                    (np.arange(m) % 2).astype(np.uint8), K @ x, rng.standard_normal(n), np.zeros(n), np.ones(n))


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("longest", [3000, 40000])
def test_steps_equal_the_row_binned_ones(prec, transpose, longest):
    """One LP per handle takes the two passes, the same LP in a batch the
    row-binned sweeps: equal iterates, averages, gradients and
    residuals.  With a row too
    long for a window its segment stays row-binned on both."""
    import paper_2508_16806_amd as pd

    lp = _lp(300001, 1100003, 9500000, longest, 4, transpose)
    other = lpgen.planted(40, 90, 0.1, 3)
    kw = dict(precision=prec, step_size=0.01, primal_weight=1.3, unroll_capacity=6, unroll_checkpoint=1, eps=1e-12,
              max_iters=128)
    one, two = pd.Solver(lp, **kw), pd.Solver([lp, other], **kw)
    rng = np.random.default_rng(1)
    gx, gy = rng.standard_normal(lp.n), rng.standard_normal(lp.m)
    pad = lambda g, k: np.concatenate([g, np.zeros(k)])
    for s in (one, two):
        s.iterate(6, record=True)
    for a, b in zip(one.solution(which=pd.SOL_CURRENT), two.solution(which=pd.SOL_CURRENT)):
        assert np.array_equal(a, b)
    ga, gb = one.backward(gx, gy), two.backward(pad(gx, other.n), pad(gy, other.m))
    for k in ga:
        assert np.array_equal(ga[k], gb[k][:ga[k].size]), k
    r1, r2 = one.solve()[0], two.solve()[0]
    assert r1["kkt"] == r2["kkt"] and r1["iters"] == r2["iters"]
    for which in (pd.SOL_CURRENT, pd.SOL_AVERAGE):
        for a, b in zip(one.solution(which=which), two.solution(which=which)):
            assert np.array_equal(a, b)
