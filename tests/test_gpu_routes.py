"""The sweeps that the LPs of the other tests take (pdhg_get_sweeps): a test of a
kernel is one only while its LPs take it."""
import ctypes as C

import pytest

import lpgen
import test_gpu_adjoint_replay as replay
import test_gpu_small as small
import test_gpu_spread as spread
import test_gpu_tile as tile

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pd():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_16806_amd as pd

    pd.lib()
    return pd


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_small(pd, prec):
    for name, f in small.LPS.items():
        assert pd.Solver(f(), precision=prec).sweeps() == ("small", "small"), name
    big = lpgen.planted(2000, 5000, 0.006, 9)
    b = pd.Solver([small.LPS["tiny"](), big], precision=prec)
    assert [b.sweeps(i) for i in (0, 1)] == [("direct", "direct")] * 2  # a mixed batch
    assert pd.Solver(small.LPS["dense3"](), precision=prec, col_slices=2).sweeps() == ("direct", "rows")


# (primal, dual) in FP32 and in FP64
TILES = {
    "wg256": [("direct", "direct")] * 2,
    "edge64": [("tiles", "tiles")] * 2,
    "edge64+1": [("tiles", "tiles")] * 2,
    "edge32": [("tiles", "tiles"), ("tiles", "rows")],
    "edge32+1": [("tiles", "tiles"), ("tiles", "rows")],
    "tiles": [("tiles", "tiles"), ("tiles", "rows")],
    "sparse": [("rows", "tiles")] * 2,
    "rows": [("rows", "tiles")] * 2,
}


@pytest.mark.parametrize("name", sorted(TILES))
def test_tiles(pd, name):
    got = [pd.Solver(tile.LPS[name](), precision=p).sweeps() for p in ("f32", "f64")]
    assert got == TILES[name]


def test_windows(pd):
    other = lpgen.planted(40, 90, 0.1, 3)
    for transpose in (False, True):
        lp = spread._lp(300001, 1100003, 9500000, 3000, 4, transpose)
        for prec in ("f32", "f64"):
            want = ("windows", "rows") if transpose else ("rows", "windows")
            assert pd.Solver(lp, precision=prec).sweeps() == want
            assert pd.Solver([lp, other], precision=prec).sweeps() == ("rows", "rows")


def test_adjoint(pd):
    want = {"small": "small", "tall": "small", "tile": "direct", "rows": "rows"}
    for name, shape in replay.LPS.items():
        assert pd.Solver(replay._tied(*shape, seed=5)[0], precision="f64").sweeps() == (want[name],) * 2, name


def test_without_layouts_and_bad_arguments(pd):
    lps = [lpgen.planted(800, 2000, 0.008, 100 + i) for i in range(72)]
    s = pd.Solver(lps, noalloc=True, precision="f64")
    assert s.sweeps(71) == ("rows", "rows")
    s.close()
    s = pd.Solver(lpgen.tiny(3, n=5, m=3))
    v = C.c_int32(7)
    L = pd.lib()
    assert L.pdhg_get_sweeps(s.h, 0, None, None) == 0
    for inst in (-1, 1):
        assert L.pdhg_get_sweeps(s.h, inst, C.byref(v), None) == -1 and v.value == 7
    assert L.pdhg_get_sweeps(None, 0, C.byref(v), None) == -1
