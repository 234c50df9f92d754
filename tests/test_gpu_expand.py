"""Column panels in two steps (the csr_panel default): edges of its panels,
row blocks and threads.  Whole-number values and vectors make every sum exact
in any order, so results are compared bit for bit with the exact product."""
import numpy as np
import pytest

from oracle import spmv as O

pytestmark = pytest.mark.gpu

PANEL = {np.float32: 20352, np.float64: 10176}    # columns of a panel (81408 bytes of x)
BLOCK = {np.float32: 16384, np.float64: 8192}     # entries of a row block


def _matrix(rng, lengths, n):
    """Rows of the given lengths with random distinct ascending columns."""
    lengths = np.asarray(lengths, dtype=np.int64)
    rp = np.concatenate([[0], np.cumsum(lengths)])
    col = np.concatenate([np.sort(rng.choice(n, size=k, replace=False)) for k in lengths]
                         + [np.zeros(0, np.int64)]).astype(np.int32)
    return rp, col


def _check(rp, col, n, dtype, rng, kind=None, params=None, x=None):
    import torch
    from paper_1210_2536_amd.spmv import Plan
    val = rng.integers(-8, 9, size=col.size).astype(dtype)   # zeros stored among them
    x = rng.integers(-64, 65, size=n).astype(dtype) if x is None else x
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    args = (t(rp.astype(np.int32)), t(col), t(val))
    p = Plan(*args, n=n, selector="csr_panel", params=params)
    assert p.info()["params"]["panel_xcd"] == 0, "the two-step form is the default here"
    y = torch.full((rp.size - 1,), float("nan"), dtype=args[2].dtype, device="cuda")
    xd = t(x)
    p.run(xd, y)
    ok = np.isfinite(x)
    ref, _ = O.spmv_accurate(rp, col, val.astype(np.float64), np.where(ok, x, 0).astype(np.float64))
    bad = np.zeros(rp.size - 1, dtype=bool)   # rows that store a non-finite x
    if not ok.all():
        rows = np.repeat(np.arange(rp.size - 1), np.diff(rp))
        bad[rows[~ok[col]]] = True
    got = y.cpu().numpy()
    assert np.array_equal(got[~bad], ref[~bad].astype(dtype)), kind
    assert not np.isfinite(got[bad]).any()
    y2 = torch.empty_like(y)
    p.run(xd, y2)
    assert np.array_equal(y2.cpu().numpy().view(np.uint8), got.view(np.uint8))
    r2, c2, v2 = p.roundtrip()
    assert torch.equal(r2, args[0]) and torch.equal(c2, args[1])
    assert np.array_equal(v2.cpu().numpy().view(np.uint8), val.view(np.uint8))
    return p


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("dn", [-1, 0, 1])
def test_panel_edges(dtype, dn):
    W = PANEL[dtype]
    rng = np.random.default_rng([70, dn + 1])
    for n in (W + dn, 2 * W + dn, 5):
        rp, col = _matrix(rng, rng.integers(0, min(n, 40) + 1, size=700), n)
        col[rp[1:][np.diff(rp) > 0] - 1] = n - 1       # the last column of every row
        _check(rp, col, n, dtype, rng, f"n={n}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("kind", ["full", "full+1", "ones", "empty", "one_row", "thread_rows",
                                  "mixed", "ragged"])
def test_row_block_edges(dtype, kind):
    rng = np.random.default_rng(71)
    E, n = BLOCK[dtype], 50_001
    lengths = {
        "full": [64] * (2 * E // 64),                   # blocks without padding
        "full+1": [64] * (E // 64) + [1],
        "ones": [1] * (2 * E + 3),                      # a row per entry
        "empty": [0] * 5000 + [3] + [0] * 5000,
        "one_row": [1000],
        "thread_rows": [16, 8, 16, 8, 7, 9, 15, 17] * 600,
        "mixed": rng.integers(0, 1025, size=200),
        "ragged": np.where(rng.random(9000) < 0.02, rng.integers(300, 1024, 9000),
                           rng.integers(0, 4, 9000)),
    }[kind]
    rp, col = _matrix(rng, lengths, n)
    _check(rp, col, n, dtype, rng, kind)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("long_lds", [0, 2, 3])
def test_rows_left_to_other_kernels(dtype, long_lds):
    """Rows above the blocks' limit, first, last and next to empty ones."""
    rng = np.random.default_rng(72)
    n = 41_000
    lengths = rng.integers(0, 30, size=3000)
    lengths[[0, 1, 17, 18, 1500, 2999]] = [1025, 0, 3000, 1024, 1100, 2000]
    rp, col = _matrix(rng, lengths, n)
    p = _check(rp, col, n, dtype, rng, params={"long_lds": long_lds} if long_lds else None)
    assert (p.info()["long_rows"] > 0) == (long_lds == 3)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
def test_non_finite_x_stays_in_its_rows(dtype):
    """Padding, empty rows and rows of other kernels multiply no x of theirs."""
    rng = np.random.default_rng(73)
    n = 30_000
    lengths = rng.integers(0, 20, size=4000)
    lengths[5] = 1500
    rp, col = _matrix(rng, lengths, n)
    x = rng.integers(-64, 65, size=n).astype(dtype)
    x[[0, 777, n - 1]] = [np.inf, np.nan, -np.inf]
    _check(rp, col, n, dtype, rng, x=x)


def test_other_forms_stay_as_asked():
    import torch
    from paper_1210_2536_amd.spmv import Plan
    rng = np.random.default_rng(74)
    rp, col = _matrix(rng, rng.integers(1, 30, size=2000), 30_000)
    val = rng.integers(-8, 9, size=col.size).astype(np.float32)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    for params, xcd in (({"panel_xcd": 1}, 1), ({"panel_xcd": 2}, 2), ({"panel_kib": 16}, 1),
                        ({"panel_direct_max": 4}, 1), (None, 0)):
        p = Plan(t(rp.astype(np.int32)), t(col), t(val), n=30_000, selector="csr_panel",
                 params=params)
        got = p.info()["params"]
        assert got["panel_xcd"] == xcd
        # a plan made again from its recorded parameters has the same form
        q = Plan(t(rp.astype(np.int32)), t(col), t(val), n=30_000, selector="csr_panel",
                 params=got)
        assert q.info()["params"] == got


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("panels", [1, 3, 65, 260, 900])
def test_runs_of_panels(dtype, panels):
    """A row block's runs of xe per panel: empty ones, ones of a lane, ones
    longer than the lanes that copy them, and more than are copied at once."""
    rng = np.random.default_rng([75, panels])
    W = PANEL[dtype]
    n = panels * W - 7
    rows = []
    for r in range(2500):
        a = rng.integers(0, min(n, W), size=r % 7)           # the first panel
        b = rng.integers(0, panels, size=r % 13) // 3 * 3 * W + rng.integers(0, W, size=r % 13)
        rows.append(np.unique(np.concatenate([a, b[b < n]])))
    rp = np.concatenate([[0], np.cumsum([c.size for c in rows])])
    _check(rp, np.concatenate(rows).astype(np.int32), n, dtype, rng, f"panels={panels}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
def test_storage_cap_between_the_forms(dtype):
    """A cap that only the XCD panels fit leaves the two steps unbuilt."""
    import torch
    from paper_1210_2536_amd import capi as C
    from paper_1210_2536_amd.spmv import Plan
    rng = np.random.default_rng(76)
    elt = np.dtype(dtype).itemsize
    m, n, k = 20_000, 600_000, 100
    col = np.sort(rng.integers(0, n // k, size=(m, k)) + np.arange(k) * (n // k), axis=1)
    rp = torch.arange(0, m * k + 1, k, dtype=torch.int32, device="cuda")
    ci = torch.from_numpy(col.reshape(-1).astype(np.int32)).cuda()
    va = torch.from_numpy(rng.integers(-8, 9, size=m * k).astype(dtype)).cuda()
    x = torch.from_numpy(rng.integers(-64, 65, size=n).astype(dtype)).cuda()
    rest = [q for q in C.KERNELS if q != "csr_panel"]
    xcd_bytes = m * k * (elt + 4) + 16 * (m + 1) * 4 + 16 * m * elt
    y = []
    for cap, form in ((xcd_bytes, 1), (100 << 20, 0)):
        p = Plan(rp, ci, va, n=n, selector="exhaustive", disable=rest, mem_cap=cap)
        i = p.info()
        assert i["kernel_name"] == "csr_panel" and i["params"]["panel_xcd"] == form
        y.append(p.run(x))
    assert torch.equal(y[0], y[1])   # whole numbers: exact in any order
