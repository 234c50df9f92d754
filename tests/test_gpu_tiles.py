"""Long rows by x-panel tiles at the edges of the tile kernel: panels, passes
of 16384 (8192 float64) entries, threads of 16 (8), rows without entries in a
panel, rows that fill a panel.  Whole-number data, so results are compared
bit for bit with the exact product."""
import numpy as np
import pytest

from oracle import spmv as O

pytestmark = pytest.mark.gpu

PANEL = {np.float32: 20352, np.float64: 10176}
PASS = {np.float32: 16384, np.float64: 8192}


def _rows(rng, kind, W, E):
    """(columns of each row, n)"""
    pick = lambda k, lo, hi: np.sort(rng.choice(np.arange(lo, hi), size=k, replace=False))  # noqa: E731
    n = 3 * W + 5
    if kind == "pass":            # panel 0: segments that fill a pass to the entry
        return [pick(E // 4, 0, W) for _ in range(4)] + [pick(E // 2, 0, W)] * 2 + \
            [pick(300, 0, n)], n
    if kind == "pass+1":
        return [pick(E // 4, 0, W) for _ in range(4)] + [pick(301, 0, n)] * 3, n
    if kind == "dense":           # every column of every panel
        return [np.arange(n), pick(400, W, 2 * W), np.arange(n)], n
    if kind == "one_panel":       # the other panels hold no entry of any row
        return [pick(300 + i, 2 * W, 3 * W) for i in range(40)], n
    if kind == "threads":         # segments that end on and beside thread edges
        return [np.concatenate([pick(k, 0, W), pick(500 - k, W, 2 * W)])
                for k in (16, 8, 15, 17, 1, 32, 31, 33) * 30], n
    if kind == "edges":           # first and last column of every panel
        e = np.unique(np.r_[0, W - 1, W, 2 * W - 1, 2 * W, 3 * W - 1, 3 * W, n - 1])
        return [np.union1d(e, pick(400, 0, n)) for _ in range(50)], n
    return [pick(int(k), 0, n) for k in rng.integers(257, 6000, size=600)], n   # many


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("kernel", ["csr_adaptive", "csr_panel"])
@pytest.mark.parametrize("kind", ["pass", "pass+1", "dense", "one_panel", "threads", "edges",
                                  "many"])
def test_tile_edges(kind, kernel, dtype):
    import torch
    from paper_1210_2536_amd.spmv import Plan
    rng = np.random.default_rng([75, len(kind)])
    W, E = PANEL[dtype], PASS[dtype]
    rows, n = _rows(rng, kind, W, E)
    short = [np.sort(rng.choice(n, size=k, replace=False)) for k in rng.integers(0, 20, size=200)]
    order = rng.permutation(len(rows) + len(short))
    allr = [(rows + short)[i] for i in order]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in allr])])
    col = np.concatenate(allr).astype(np.int32)
    val = rng.integers(-4, 5, size=col.size).astype(dtype)
    x = rng.integers(-8, 9, size=n).astype(dtype)
    x[[1, W + 1]] = np.inf        # padding must not multiply it into rows without it
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    p = Plan(t(rp.astype(np.int32)), t(col), t(val), n=n, selector=kernel,
             params={"long_lds": 3, "tile_row_min": 256})
    info = p.info()
    assert info["params"]["long_lds"] == 3 and info["long_rows"] == len(rows)
    xd = t(x)
    y = torch.full((rp.size - 1,), float("nan"), dtype=xd.dtype, device="cuda")
    p.run(xd, y)
    ok = np.isfinite(x)
    ref, _ = O.spmv_accurate(rp, col, val.astype(np.float64), np.where(ok, x, 0).astype(np.float64))
    r = np.repeat(np.arange(rp.size - 1), np.diff(rp))
    bad = np.zeros(rp.size - 1, dtype=bool)
    bad[r[~ok[col]]] = True
    got = y.cpu().numpy()
    assert np.array_equal(got[~bad], ref[~bad].astype(dtype)), kind
    assert not np.isfinite(got[bad]).any()
    y2 = torch.empty_like(y)
    p.run(xd, y2)
    assert np.array_equal(y2.cpu().numpy().view(np.uint8), got.view(np.uint8))
