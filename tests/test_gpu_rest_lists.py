"""Operators with tiled (windowed) and row-binned rows: the row-binned sweeps walk a
list of their own blocks."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _lps():
    return [
        lpgen.planted(3001, 2003, 0.02, 8, ge_frac=0.5),  # tiled
        lpgen.planted(400, 450, 0.5, 1),  # over local columns: row bins
        lpgen.from_dense(np.zeros((0, 6)), [], [], np.linspace(-1, 1, 6), np.zeros(6), np.ones(6)),  # no rows
        lpgen.planted(90000, 12000, 0.0012, 6, ge_frac=0.5),  # the dual sweep tiled only
        lpgen.planted(300, 350, 0.6, 2, ge_frac=0.5),  # row bins
        lpgen.planted(700, 3000, 0.012, 3),  # tiled
    ]


@pytest.mark.parametrize("budget", [0, 1, 20_000_000])
@pytest.mark.parametrize("remap", [0, 1])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_batch_equals_solo(prec, remap, budget):
    """All at once, one at a time and a few at a time, with restarts and averages,
    fixed steps and gradients: each as alone, bit for bit."""
    import paper_2508_16806_amd as pd

    lps = _lps()
    kw = dict(precision=prec, xcd_remap=remap, max_iters=192, unroll_capacity=5, unroll_checkpoint=1)
    b = pd.Solver(lps, batch_resident_bytes=budget, **kw)
    kinds = [b.sweeps(i) for i in range(len(lps))]
    assert kinds[1] == kinds[4] == ("rows", "rows") and "rows" not in kinds[0] and kinds[3][0] == "rows" != kinds[3][1]
    rb = b.solve()
    got = [b.solution(inst=i) for i in range(len(lps))]
    b.iterate(5, record=True)
    gx, gy = np.ones(sum(p.n for p in lps)), np.ones(sum(p.m for p in lps))
    gb, at, am = b.backward(gx, gy), 0, 0
    for i, lp in enumerate(lps):
        s = pd.Solver(lp, **kw)
        r = s.solve()[0]
        assert (rb[i]["iters"], rb[i]["status"], rb[i]["restarts"]) == (r["iters"], r["status"], r["restarts"])
        for u, v in zip(got[i], s.solution()):
            np.testing.assert_array_equal(u, v, err_msg=str(i))
        s.iterate(5, record=True)
        g = s.backward(np.ones(lp.n), np.ones(lp.m))
        for key, want in g.items():
            k = am if key in ("rhs", "y0") else at
            np.testing.assert_array_equal(gb[key][k:k + want.size], want, err_msg=f"{i} {key}")
        at, am = at + lp.n, am + lp.m


@pytest.mark.parametrize("slices", [0, 2])
def test_sliced_rows_beside_tiles(slices):
    """An LP with sliced rows beside tiled ones: as alone, bit for bit."""
    import paper_2508_16806_amd as pd

    lps = [lpgen.planted(700, 3000, 0.004, 3), lpgen.config2(7, m=3000, n=6000, kmax=2000), lpgen.planted(400, 450, 0.5, 1)]
    kw = dict(precision="f64", max_iters=192, col_slices=4, col_slices_t=slices)
    b = pd.Solver(lps, **kw)
    assert b.sweeps(0)[1] != "rows" == b.sweeps(1)[1]
    b.solve()
    for i, lp in enumerate(lps):
        s = pd.Solver(lp, **kw)
        s.solve()
        for u, v in zip(b.solution(inst=i), s.solution()):
            np.testing.assert_array_equal(u, v, err_msg=str(i))
