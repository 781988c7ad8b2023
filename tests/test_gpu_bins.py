"""The library's own row-length limits: rows at and beside every limit."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24
DEFAULT = [8, 16, 32, 64, 128, 256, 512, 0]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("transpose", [False, True])
def test_rows_at_the_limits(orc, prec, transpose):
    """Rows (columns) of 0, 1, 7, 8, 9, ... 513 entries, too few entries for
    the sweeps that gather from LDS and vectors too long for the
    one-workgroup iteration: the oracle's iterates, and bit for bit those of the
    same limits given as options.  20 FP32 steps: each rounds data, matrix
    and iterate (8 roundings of 2^-24 of the largest entry), and a step does
    not enlarge earlier errors in the omega-weighted norm (factor 1.3 either
    way between x and y)."""
    import scipy.sparse as sp

    import paper_2508_16806_amd as pd

    lens = [0, 1] + [b + d for b in DEFAULT[:7] for d in (-1, 0, 1)]
    rng = np.random.default_rng(5)
    R, N = 40 * len(lens), 60000
    rows = np.repeat(np.arange(R), np.tile(lens, 40))
    cols = np.concatenate([rng.choice(N, k, replace=False) for k in np.tile(lens, 40)])
    K = sp.csr_matrix((rng.standard_normal(rows.size), (rows, cols)), shape=(R, N))
    if transpose:
        K = K.T.tocsr()
    K.sort_indices()
    m, n = K.shape
    x = rng.uniform(0, 1, n)
    lp = lpgen.LP(n, m, K.indptr.astype(np.int64), K.indices.astype(np.int32), K.data,
                  (np.arange(m) % 2).astype(np.uint8), K @ x, rng.standard_normal(n), np.zeros(n), np.ones(n))
    o = orc.Oracle(lp)
    rho, kap = o.ruiz(10)
    eta, omega, k = 0.9 / pd.Solver(lp, precision="f64").info()["knorm"], 1.3, 20
    got = []
    for lim in (None, DEFAULT):
        kw = {} if lim is None else dict(bin_len_dual=lim, bin_len_primal=lim)
        s = pd.Solver(lp, precision=prec, step_size=eta, primal_weight=omega, **kw)
        s.iterate(k)
        got.append(s.solution(which=pd.SOL_CURRENT))
    x0 = np.clip(np.zeros(n), lp.l / kap, lp.u / kap)
    xs, ys = o.steps(x0, np.zeros(m), eta / omega, eta * omega, k, ruiz_iters=10)
    ref = (np.clip(kap * xs, lp.l, lp.u), rho * ys)
    scale, size = 1 + max(np.abs(v).max() for v in ref), n + m
    for a, c, b in zip(got[0], got[1], ref):
        assert np.array_equal(a, c)
        if prec == "f64":
            np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * scale)
        else:
            assert np.linalg.norm(a - b) <= 1.3 ** 2 * k * 8 * U32 * scale * np.sqrt(size)
