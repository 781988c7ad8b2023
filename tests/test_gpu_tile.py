"""The sweeps that gather from LDS (tile.hip): the row-binned sweeps' iteration
up to FP64 summation order."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu
U32 = 2.0 ** -24


@pytest.fixture(scope="module")
def pd():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_16806_amd as pd

    pd.lib()
    return pd


# the widest single tile (FP64: 16,380 columns, FP32: 32,764) and one more column
# (two tiles in one precision), several tiles, rows of few entries with an
# operator too wide for its size beside it (row-binned sweeps), more rows than a
# block takes, a size that takes workgroups of 256 lanes, and a small LP and one
# of middle size (neither is tiled)
LPS = {
    "wg256": lambda: lpgen.planted(3001, 2003, 0.02, 8, ge_frac=0.5),
    "edge64": lambda: lpgen.planted(11000, 16380, 0.015, 1, ge_frac=0.5),
    "edge64+1": lambda: lpgen.planted(11001, 16381, 0.015, 2, ge_frac=1.0),
    "edge32": lambda: lpgen.planted(5500, 32764, 0.015, 3, ge_frac=0.5),
    "edge32+1": lambda: lpgen.planted(5500, 32765, 0.015, 4),
    "tiles": lambda: lpgen.planted(5001, 70001, 0.014, 5, ge_frac=0.5),
    "sparse": lambda: lpgen.planted(90000, 12000, 0.0012, 6, ge_frac=0.5),
    "rows": lambda: lpgen.planted(400000, 10000, 0.0005, 7, ge_frac=0.5),
}
SMALL = {"small": lambda: lpgen.planted(120, 301, 0.05, 20), "middle": lambda: lpgen.planted(3000, 7001, 0.01, 21)}


def _steps(orc, pd, lp, prec, k):
    o = orc.Oracle(lp)
    rho, kap = o.ruiz(10)
    eta, omega = 0.9 / pd.Solver(lp, precision="f64").info()["knorm"], 1.3
    s = pd.Solver(lp, precision=prec, step_size=eta, primal_weight=omega)
    s.iterate(k)
    x0 = np.clip(np.zeros(lp.n), lp.l / kap, lp.u / kap)
    xs, ys = o.steps(x0, np.zeros(lp.m), eta / omega, eta * omega, k, ruiz_iters=10)
    return s.solution(which=pd.SOL_CURRENT), (np.clip(kap * xs, lp.l, lp.u), rho * ys)


@pytest.mark.parametrize("name", sorted(LPS))
def test_steps_f64(orc, pd, name):
    for a, b in zip(*_steps(orc, pd, LPS[name](), "f64", 40)):
        np.testing.assert_allclose(a, b, rtol=1e-9, atol=1e-9 * (1 + np.abs(b).max()))


@pytest.mark.parametrize("name", sorted(LPS))
def test_steps_f32(orc, pd, name):
    """20 steps: each rounds data, matrix and iterate (8 roundings of 2^-24 of
    the largest entry), and a step does not enlarge earlier errors in the
    omega-weighted norm (factor 1.3 either way between x and y)."""
    got, ref = _steps(orc, pd, LPS[name](), "f32", 20)
    scale = 1 + max(np.abs(v).max() for v in ref)
    n = sum(v.size for v in ref)
    for a, b in zip(got, ref):
        assert np.linalg.norm(a - b) <= 1.3 ** 2 * 20 * 8 * U32 * scale * np.sqrt(n)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("budget", [0, 1])
def test_batch_equals_solo(pd, prec, budget):
    """Tiled, part-tiled and untiled instances in one handle (their vectors then
    start at any alignment), all at once and admitted one at a time: each bit
    for bit as alone."""
    lps = [SMALL["small"](), LPS["edge64+1"](), SMALL["middle"](), LPS["wg256"](), LPS["sparse"]()]
    kw = dict(precision=prec, max_iters=192)
    b = pd.Solver(lps, batch_resident_bytes=budget, **kw)
    rb = b.solve()
    for i, lp in enumerate(lps):
        s = pd.Solver(lp, **kw)
        r = s.solve()[0]
        assert (rb[i]["iters"], rb[i]["status"], rb[i]["restarts"]) == (r["iters"], r["status"], r["restarts"])
        for u, v in zip(b.solution(inst=i), s.solution()):
            np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("name", ["wg256", "sparse"])
def test_adjoint(orc, pd, name):
    """Clip masks recorded by the replay."""
    lp = LPS[name]()
    o = orc.Oracle(lp)
    kn, _ = o.power_norm(10, max_iters=5000, tol=1e-10)
    eta, omega, K = 0.8 / kn, 1.7, 12
    s = pd.Solver(lp, precision="f64", step_size=eta, primal_weight=omega, unroll_capacity=K, unroll_checkpoint=5)
    rng = np.random.default_rng(1)
    gx, gy = rng.standard_normal(lp.n), rng.standard_normal(lp.m)
    x0 = rng.uniform(lp.l, lp.u)
    s.set_state(x0, np.zeros(lp.m))
    s.iterate(K, record=True)
    g = s.backward(gx, gy)
    go = o.unrolled_vjp(10, eta / omega, eta * omega, lp.c, lp.rhs, lp.l, lp.u, x0, np.zeros(lp.m), K, gx, gy)
    for k, key in (("c", "c"), ("rhs", "q"), ("l", "l"), ("u", "u"), ("x0", "x0"), ("y0", "y0")):
        assert np.linalg.norm(g[k] - go[key]) <= 1e-9 * (np.linalg.norm(go[key]) + 1e-30), k
