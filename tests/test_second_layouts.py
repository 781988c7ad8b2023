"""Which LPs get second layouts for their sweeps, seen from the workspace sizes
(host side)."""
import ctypes as C

import pytest

import lpgen


def _sizes(lp, **kw):
    import paper_2508_16806_amd as pd

    d = pd._Desc(lp)
    arr = (pd.LPDesc * 1)(d.desc)
    a = (C.cast(arr, C.c_void_p), 1, C.byref(pd.default_opts(**kw)))
    return pd.lib().pdhg_workspace_bytes(*a), pd.lib().pdhg_workspace_min_bytes(*a)


@pytest.mark.parametrize("G", [120, 250, 350, 500, 700, 1000, 1400])
def test_dispatch_lps_have_none(G):
    """Dispatch LPs of any size gather from shared lines (their dense rows, few among
    many short ones, hold most entries): row-binned sweeps in both precisions."""
    lp = lpgen.sced(G=G, B=max(2, 2 * G // 5))
    for prec in ("f32", "f64"):
        need, least = _sizes(lp, precision=prec)
        assert need == least > 0


@pytest.mark.parametrize("m,n,density", [(1000, 2500, 0.02), (20000, 50000, 0.002), (5000, 12500, 0.004)])
def test_random_lps_have_them(m, n, density):
    need, least = _sizes(lpgen.planted(m, n, density, 1), precision="f32")
    assert need > least > 0
