"""The adjoint's masks are those of the recorded steps, also where a clip is
decided by the last bit of a row's sum."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _tied(m, n, density, seed):
    """An LP and a start (x = 0 = l, y) whose reduced costs c - K'y are zero up to
    the rounding of their sums: whether a step leaves x_j at its bound depends on
    the order in which column j is added.  Equality rows with rhs 0, so y moves by
    such roundings only."""
    rng = np.random.default_rng(seed)
    A = np.where(rng.random((m, n)) < density, rng.standard_normal((m, n)), 0.0)
    y = rng.standard_normal(m)
    return lpgen.from_dense(A, np.ones(m), np.zeros(m), A.T @ y, np.zeros(n), np.ones(n)), A, y


# rows of the two sweeps by tiles, by row bins and in one workgroup
LPS = {"small": (200, 500, 0.1), "tall": (800, 60, 0.3), "tile": (3000, 4000, 0.01), "rows": (600, 700, 0.5)}


@pytest.mark.parametrize("C", [16, 3, 1])
@pytest.mark.parametrize("name", sorted(LPS))
def test_masks_are_the_recorded_steps(name, C):
    """K recorded steps end bit for bit where K single steps end, whose points
    give every step's clip (x = 0 exactly at the bound, an untouched y: no
    scaling, FP64).  The reverse recursion with these clips, in numpy, against the
    library: sums of at most K terms over at most 800 entries of order 1, so
    1e-11; one clip taken otherwise changes dL/dc_j by tau |g_j|."""
    import paper_2508_16806_amd as pd

    lp, A, y0 = _tied(*LPS[name], seed=5)
    K, tau, sigma = 16, 0.01, 0.02
    kw = dict(precision="f64", ruiz_iters=0, step_size=np.sqrt(tau * sigma), primal_weight=np.sqrt(sigma / tau))
    s = pd.Solver(lp, **kw)
    tau, sigma = s.info()["tau"], s.info()["sigma"]
    s.set_state(np.zeros(lp.n), y0)
    pts = []
    for _ in range(K):
        s.iterate(1)
        pts.append(s.solution(which=pd.SOL_CURRENT))
    inside = [(x > 0.0) & (x < 1.0) for x, _ in pts]
    assert 0.2 < np.mean(inside[0]) < 0.8  # the ties are there
    r = pd.Solver(lp, unroll_capacity=K, unroll_checkpoint=C, **kw)
    r.set_state(np.zeros(lp.n), y0)
    r.iterate(K, record=True)
    for a, b in zip(r.solution(which=pd.SOL_CURRENT), pts[-1]):
        np.testing.assert_array_equal(a, b)
    rng = np.random.default_rng(1)
    gx, gy = rng.standard_normal(lp.n), rng.standard_normal(lp.m)
    ax, ay, gc, gl = gx.copy(), gy.copy(), np.zeros(lp.n), np.zeros(lp.n)
    for t in range(K - 1, -1, -1):
        axb = -sigma * (A.T @ ay)
        g = ax + 2.0 * axb
        v = np.where(inside[t], g, 0.0)
        gc -= tau * v
        gl += np.where(pts[t][0] <= 0.0, g, 0.0)
        ay = ay + tau * (A @ v)
        ax = v - axb
    for _ in range(2):  # the first pass may have replaced the masks the recording kept
        out = r.backward(gx, gy)
        for key, want in (("c", gc), ("l", gl), ("x0", ax), ("y0", ay)):
            np.testing.assert_allclose(out[key], want, rtol=0, atol=1e-11 * (1 + np.abs(want).max()), err_msg=key)


@pytest.mark.parametrize("C", [16, 2])
def test_batch_equals_solo(C):
    """Small, tiled and row-binned LPs with ties in one handle: points and gradients
    of each as alone, bit for bit."""
    import paper_2508_16806_amd as pd

    parts = [_tied(*LPS[k], seed=5) for k in ("small", "tile", "rows", "tall")]
    kw = dict(precision="f64", ruiz_iters=0, step_size=0.01, primal_weight=1.4, unroll_capacity=16, unroll_checkpoint=C)
    rng = np.random.default_rng(2)
    g = [(rng.standard_normal(lp.n), rng.standard_normal(lp.m)) for lp, _, _ in parts]

    def adjoint(sel):
        s = pd.Solver([parts[i][0] for i in sel], **kw)
        for b, i in enumerate(sel):
            s.set_state(np.zeros(parts[i][0].n), parts[i][2], inst=b)
        s.iterate(16, record=True)
        pts = [s.solution(inst=b, which=pd.SOL_CURRENT) for b in range(len(sel))]
        return pts, s.backward(np.concatenate([g[i][0] for i in sel]), np.concatenate([g[i][1] for i in sel]))

    pts, grads = adjoint(range(len(parts)))
    at = {"n": 0, "m": 0}
    for i, (lp, _, _) in enumerate(parts):
        p1, g1 = adjoint([i])
        for u, v in zip(pts[i], p1[0]):
            np.testing.assert_array_equal(u, v)
        for key, want in g1.items():
            dim = "m" if key in ("rhs", "y0") else "n"
            np.testing.assert_array_equal(grads[key][at[dim]:at[dim] + want.size], want, err_msg=f"{i} {key}")
        at["n"] += lp.n
        at["m"] += lp.m
