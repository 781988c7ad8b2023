"""The adjoint's held and replayed clip masks: every split of the tape gives the
same gradients."""
import numpy as np
import pytest

import lpgen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name", ["rows", "lds", "small"])
def test_gradients_do_not_depend_on_the_checkpoints(prec, name):
    """K steps with checkpoints so far apart that every mask is held, against
    spacings that hold all, all but one or a few of the masks or none of a small
    LP's: bit for bit (the same sweeps make the masks), and again from the same
    tape, whose masks the first pass has replaced, and after unrecorded steps."""
    import paper_2508_16806_amd as pd

    lp = {"rows": lambda: lpgen.planted(3000, 7001, 0.01, 21, ge_frac=0.5),
          "lds": lambda: lpgen.planted(3001, 2003, 0.02, 8, ge_frac=0.5),
          "small": lambda: lpgen.planted(120, 301, 0.05, 20, ge_frac=0.5)}[name]()
    K = 41
    rng = np.random.default_rng(3)
    x0, y0 = rng.uniform(0, 1, lp.n), rng.standard_normal(lp.m)
    gx, gy = rng.standard_normal(lp.n), rng.standard_normal(lp.m)
    ref = None
    for C in (K, 11, 10, 5, 3, 1):
        s = pd.Solver(lp, precision=prec, unroll_capacity=K, unroll_checkpoint=C)
        s.set_state(x0, y0)
        s.iterate(K, record=True)
        out = [s.backward(gx, gy)]
        s.iterate(3)
        out.append(s.backward(gx, gy))
        # a shorter tape in place of the first
        s.set_state(x0, y0)
        s.iterate(7, record=True)
        short = s.backward(gx, gy)
        if ref is None:
            ref, ref7 = out[0], short
            assert any(np.count_nonzero(ref[k]) for k in ("l", "u"))  # some masks are set
        for g, want in ((out[0], ref), (out[1], ref), (short, ref7)):
            for key in ref:
                assert np.array_equal(g[key], want[key]), (C, key)
