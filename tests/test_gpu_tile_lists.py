"""Block lists of the tiled sweeps: batches whose instances enter one after another,
and batches of more instances than the list kernel's workgroup has lanes."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


def _check(lps, which, **kw):
    import paper_2508_16806_amd as pd

    b = pd.Solver(lps, **kw)
    rb = b.solve()
    for i in which:
        s = pd.Solver(lps[i], **{k: v for k, v in kw.items() if k != "batch_resident_bytes"})
        r = s.solve()[0]
        assert (rb[i]["iters"], rb[i]["status"], rb[i]["restarts"]) == (r["iters"], r["status"], r["restarts"])
        for u, v in zip(b.solution(inst=i), s.solution()):
            np.testing.assert_array_equal(u, v, err_msg=str(i))


@pytest.mark.parametrize("budget", [0, 1, 3_000_000, 20_000_000])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_budgets(prec, budget):
    """All at once, one at a time and a few at a time: launches of as many
    workgroups as blocks run at most.  Each instance as alone, bit for bit."""
    lps = [lpgen.planted(700 + 300 * i, 2000 + 700 * i, 0.012, i, ge_frac=0.5) for i in range(9)]
    _check(lps, range(len(lps)), precision=prec, max_iters=192, batch_resident_bytes=budget)


@pytest.mark.parametrize("budget", [0, 400_000])
def test_more_instances_than_lanes(budget):
    """1,100 small LPs take the tiles beside one that is not small."""
    lps = [lpgen.tiny(i, n=4 + i % 9, m=2 + i % 5) for i in range(1100)]
    lps.insert(500, lpgen.planted(2000, 5000, 0.006, 9, ge_frac=0.5))
    _check(lps, [0, 1, 499, 500, 501, 1022, 1023, 1024, 1025, 1100], precision="f32", max_iters=128,
           batch_resident_bytes=budget)
