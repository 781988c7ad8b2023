"""Fishnet sweeps at the row lengths where a task changes its kind."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("P", [2, 8, 32, 64])
def test_row_lengths(orc, P, transpose):
    """Rows (columns) of 0 to 9 entries and around the lengths that take a
    workgroup (128) and that are cut (1024), on every number of lanes per point;
    FP64: the oracle's kept points, and its gaps and survivor to 1e-9."""
    import scipy.sparse as sp

    import paper_2508_16806_amd as pd

    lens = list(range(10)) + [31, 32, 33, 127, 128, 129, 1023, 1024, 1025, 2049]
    rng = np.random.default_rng(7)
    rows = np.repeat(np.arange(len(lens)), lens)
    cols = np.concatenate([rng.choice(2500, k, replace=False) for k in lens])
    K = sp.csr_matrix((rng.standard_normal(rows.size), (rows, cols)), shape=(len(lens), 2500))
    if transpose:
        K = K.T.tocsr()
    K.sort_indices()
    m, n = K.shape
    x = rng.uniform(0, 1, n)
    lp = lpgen.LP(n, m, K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data,
                  (np.arange(m) % 2).astype(np.uint8), K @ x, rng.standard_normal(n), np.zeros(n), np.ones(n))
    s = pd.Solver(lp, precision="f64", fishnet_points=P)
    info = s.info()
    G, wraw = lpgen.fishnet_draws(n, P, seed=3)
    out = s.fishnet(P, 6, G=G, wraw=wraw)
    xs, ys = s.solution(which=pd.SOL_CURRENT)
    xo, yo, gaps, keep = orc.Oracle(lp).fishnet(10, info["eta"], info["omega"], info["knorm"], P, 6, G, wraw)
    assert [list(k)[:len(o)] for k, o in zip(out["keep"], keep)] == [list(o) for o in keep]
    live = gaps != 0.0
    np.testing.assert_allclose(out["gaps"][live], gaps[live], rtol=1e-8, atol=1e-12)
    for a, b in ((xs, xo), (ys, yo)):
        assert np.linalg.norm(a - b) <= 1e-9 * (1.0 + np.linalg.norm(b))
