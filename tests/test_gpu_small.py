"""Fixed-step iterations of small LPs in one workgroup (small.hip): the
iteration of the sweeps that gather from LDS (tile.hip), bit for bit."""
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


# edges: fewer rows than a wavefront, task remainders, rows over many lanes
# (a few rows of ~470 entries), empty rows and columns, each level of what
# fits in LDS (FP64 / FP32), no rows at all
LPS = {
    "tiny": lambda: lpgen.tiny(3, n=5, m=3),
    "m63n65": lambda: lpgen.planted(63, 65, 0.1, 1, ge_frac=0.5),
    "m64n64": lambda: lpgen.planted(64, 64, 0.2, 2),
    "dense3": lambda: lpgen.planted(3, 520, 0.9, 3, ge_frac=0.5),
    "sparse": lambda: lpgen.planted(300, 1100, 0.002, 4, ge_frac=0.3),
    "n1025": lambda: lpgen.planted(511, 1025, 0.01, 5, ge_frac=1.0),
    "large": lambda: lpgen.planted(1003, 2501, 0.005, 6, ge_frac=0.5),
    "wide": lambda: lpgen.planted(200, 5000, 0.01, 7),
}


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
@pytest.mark.parametrize("k,tol", [(2, 1e-12), (600, 1e-9)])  # 600: more steps than a launch takes
def test_steps_f64(orc, pd, name, k, tol):
    for a, b in zip(*_steps(orc, pd, LPS[name](), "f64", k)):
        np.testing.assert_allclose(a, b, rtol=tol, atol=tol * (1 + np.abs(b).max(initial=0)))


@pytest.mark.parametrize("name", sorted(LPS))
def test_steps_f32(orc, pd, name):
    """20 steps: each rounds data, matrix and iterate (8 roundings of 2^-24 of
    the largest entry), and a step does not enlarge earlier errors in the
    omega-weighted norm (factor 1.3 either way between x and y)."""
    got, ref = _steps(orc, pd, LPS[name](), "f32", 20)
    scale = 1 + max(np.abs(v).max(initial=0) for v in ref)
    n = sum(v.size for v in ref)
    for a, b in zip(got, ref):
        assert np.linalg.norm(a - b) <= 1.3 ** 2 * 20 * 8 * U32 * scale * np.sqrt(n)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("bins", [0, 2, 16])
def test_equals_the_sweeps(pd, prec, bins):
    """A batch with one LP too large for small.hip takes tile.hip: every small
    LP beside it has the bits it has alone.  Also with other row-length bins,
    whose rows have other lanes there."""
    lps = [f() for _, f in sorted(LPS.items())] + [lpgen.planted(2000, 5000, 0.006, 9)]
    kw = dict(precision=prec, max_iters=640, detect_infeas=1)
    if bins:
        kw["bin_len_dual"] = kw["bin_len_primal"] = [bins << k for k in range(6)] + [2048, 0]
    b = pd.Solver(lps, batch_resident_bytes=0, **kw)
    rb = b.solve()
    for i, lp in enumerate(lps):
        s = pd.Solver(lp, **kw)
        r = s.solve()[0]
        assert (rb[i]["iters"], rb[i]["status"], rb[i]["restarts"]) == (r["iters"], r["status"], r["restarts"])
        for u, v in zip(b.solution(inst=i), s.solution()):
            np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("budget", [0, 1])
def test_small_batch_equals_solo(pd, budget):
    """Small instances in one handle, all at once and admitted one at a time."""
    lps = [LPS["n1025"](), LPS["tiny"](), LPS["m64n64"](), LPS["sparse"]()]
    kw = dict(precision="f32", max_iters=640)
    b = pd.Solver(lps, batch_resident_bytes=budget, **kw)
    b.solve()
    for i, lp in enumerate(lps):
        s = pd.Solver(lp, **kw)
        s.solve()
        for u, v in zip(b.solution(inst=i), s.solution()):
            np.testing.assert_array_equal(u, v)


def test_noalloc_without_layouts(pd):
    """A batch whose workspace fits the fixed array only without the second
    layouts is still accepted, and takes the row-binned sweeps: the same
    iteration, row sums in another FP64 order (64 steps, as test_steps_f64)."""
    lps = [lpgen.planted(800, 2000, 0.008, 100 + i) for i in range(72)]
    kw = dict(precision="f64", max_iters=64)
    s = pd.Solver(lps, noalloc=True, **kw)
    a = pd.Solver(lps, **kw)
    assert a.info()["workspace_bytes"] > 64 << 20
    s.solve(), a.solve()
    for i in (0, 71):
        for u, v in zip(s.solution(inst=i), a.solution(inst=i)):
            np.testing.assert_allclose(u, v, rtol=1e-9, atol=1e-9 * (1 + np.abs(v).max()))
    s.close()
