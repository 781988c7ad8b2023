"""Workspaces without the sweeps' second layouts: what pdhg_setup takes and refuses."""
import ctypes as C

import numpy as np
import pytest

import lpgen


def _args(pd, lps, **kw):
    d = [pd._Desc(lp) for lp in lps]
    arr = (pd.LPDesc * len(lps))(*[q.desc for q in d])
    return C.cast(arr, C.c_void_p), len(lps), C.byref(pd.default_opts(**kw)), (d, arr)


LPS = {
    "small": [lpgen.planted(200, 500, 0.02, 1)],
    "tiles": [lpgen.planted(3001, 2003, 0.02, 8, ge_frac=0.5)],
    "batch": [lpgen.planted(3001, 2003, 0.02, 8, ge_frac=0.5), lpgen.tiny(3, n=5, m=3)],
    "local": [lpgen.planted(600, 700, 0.5, 2)],  # row bins: no second layout
}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(LPS))
def test_sizes(name, prec):
    import paper_2508_16806_amd as pd

    p, n, o, keep = _args(pd, LPS[name], precision=prec)
    need, least = pd.lib().pdhg_workspace_bytes(p, n, o), pd.lib().pdhg_workspace_min_bytes(p, n, o)
    assert 0 < least <= need and (least == need) == (name == "local")


@pytest.mark.gpu
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(LPS))
def test_setup_takes_the_least(name, prec, monkeypatch):
    """Set up in exactly pdhg_workspace_min_bytes, and through a Solver whose first
    allocation fails: row-binned sweeps, the points of the full workspace up to the
    order of the sums (64 FP64 steps: 1e-9, as the sweeps' own tests; FP32 iterates:
    64 roundings of 2^-24, factor 8).  Less than the least (sizes are rounded to 256 bytes) is refused."""
    import torch

    import paper_2508_16806_amd as pd

    lps, kw = LPS[name], dict(precision=prec, max_iters=64, use_restarts=0)
    p, n, o, keep = _args(pd, lps, **kw)
    L = pd.lib()
    full = pd.Solver(lps, **kw)
    least = L.pdhg_workspace_min_bytes(p, n, o)
    ws = torch.empty(least, dtype=torch.uint8, device="cuda")
    h = C.c_void_p()
    assert L.pdhg_setup(p, n, o, ws.data_ptr(), least - 256, None, C.byref(h)) == pd.ERR_NOMEM and not h.value
    assert "workspace too small" in L.pdhg_last_error().decode()
    assert L.pdhg_setup(p, n, o, ws.data_ptr(), least, None, C.byref(h)) == 0
    L.pdhg_destroy(h)
    real, calls = torch.empty, []

    def empty(size, *a, **k):
        calls.append(size)
        if len(calls) == 1:
            raise torch.OutOfMemoryError("no memory")
        return real(size, *a, **k)

    monkeypatch.setattr(torch, "empty", empty)
    s = pd.Solver(lps, **kw)
    monkeypatch.undo()
    assert calls == [L.pdhg_workspace_bytes(p, n, o), least] and s.info()["workspace_bytes"] <= least
    assert all(s.sweeps(i) == ("rows", "rows") for i in range(n))
    full.solve(), s.solve()
    tol = 1e-9 if prec == "f64" else 64 * 8 * 2.0 ** -24
    for i in range(n):
        for a, b in zip(s.solution(inst=i), full.solution(inst=i)):
            np.testing.assert_allclose(a, b, rtol=tol, atol=tol * (1 + np.abs(b).max()))
