"""The library's own row-length limits (opts.bin_len_* = 0): which of the two sets
an operator takes.  Host side: the workspace is that of the same limits as
options."""
import ctypes as C

import numpy as np
import pytest

import lpgen

LIM = {f: [f << k for k in range(6)] + [512, 0] for f in (4, 8)}


def _bytes(lp, **kw):
    import paper_2508_16806_amd as pd

    d = pd._Desc(lp)
    arr = (pd.LPDesc * 1)(d.desc)
    return pd.lib().pdhg_workspace_bytes(C.cast(arr, C.c_void_p), 1, C.byref(pd.default_opts(**kw)))


def _lp(lens, n, local=False, seed=1):
    """Rows of the given lengths over n columns in a random cyclic order (local: in
    their own), so that the columns' lengths differ by one at most."""
    lens = np.asarray(lens)
    order = np.arange(n) if local else np.random.default_rng(seed).permutation(n)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = order[np.arange(rowptr[-1]) % n].astype(np.int32)
    return lpgen.LP(n, lens.size, rowptr, col, np.ones(col.size), np.zeros(lens.size, dtype=np.uint8),
                    np.zeros(lens.size), np.ones(n), np.zeros(n), np.ones(n))


# K's row lengths, columns, options, limits of K and of K^T
CASES = {
    "short": (np.full(1000, 12), 2400, {}, 4, 4),  # columns of 5
    "columns_of_4": (np.full(1000, 12), 3000, {}, 4, 8),
    "199985": (np.full(199985 // 37, 37), 6666, {}, 4, 4),  # columns of 30
    "200022": (np.full(200022 // 37, 37), 6667, {}, 8, 8),
    "999999": (np.full(999999 // 37, 37), 33333, dict(adaptive_step=1), 4, 4),
    "1000036": (np.full(1000036 // 37, 37), 33333, dict(adaptive_step=1), 8, 8),
    "local": (np.full(13513, 37), 16666, dict(local=True), 4, 8),  # K over local columns: row bins
    "local_more": (np.full(13514, 37), 16667, dict(local=True), 8, 8),
    "local_adaptive": (np.full(13514, 37), 16667, dict(local=True, adaptive_step=1), 8, 4),
    "half_long": (np.r_[np.full(100, 30), np.full(10, 300)], 660, {}, 4, 4),  # 3,000 and 3,000 entries
    "more_long": (np.r_[np.full(100, 30), np.full(11, 300)], 700, {}, 8, 4),
    "sliced": (np.full(1000036 // 37, 37), 33333, dict(col_slices=2), 4, 8),
    "sliced_t": (np.full(1000036 // 37, 37), 33333, dict(col_slices_t=2), 8, 4),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_default_limits(name):
    lens, n, kw, dual, primal = CASES[name]
    kw = dict(kw)
    lp = _lp(lens, n, kw.pop("local", False))
    for prec in ("f32", "f64"):
        got = {(a, b): _bytes(lp, precision=prec, bin_len_dual=LIM[a], bin_len_primal=LIM[b], **kw)
               for a in LIM for b in LIM}
        assert len(set(got.values())) > 1  # the sets differ in blocks or segments
        want = {k for k, v in got.items() if v == _bytes(lp, precision=prec, **kw)}
        assert (dual, primal) in want and (12 - dual, 12 - primal) not in want, (want, got)
