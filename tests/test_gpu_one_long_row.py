"""Column panels of a matrix with a row far longer than the others: the row goes
to tiles or is cut by panels, never to a single workgroup.  Whole-number data,
so results are compared bit for bit."""
import numpy as np
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


def _matrix(m, n, k, long_rows, dtype):
    """k entries a row (at a random start, an odd step), `long_rows` {row: length}."""
    g = torch.Generator(device="cuda")
    g.manual_seed(91)
    length = torch.full((m,), k, dtype=torch.int64, device="cuda")
    for r, w in long_rows.items():
        length[r] = w
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=rp[1:])
    row = torch.repeat_interleave(length)
    pos = torch.arange(int(rp[-1]), device="cuda") - rp[row]
    step = (n - 1) // length[row]
    start = (torch.rand(m, device="cuda", generator=g, dtype=torch.float64) * (n // (2 * k)))
    col = pos * step + torch.where(length[row] == k, start.to(torch.int64)[row], 0)
    assert int(col.max()) < n
    val = torch.randint(-4, 5, (col.numel(),), device="cuda", generator=g).to(dtype)
    x = torch.randint(-8, 9, (n,), device="cuda", generator=g).to(dtype)
    # whole numbers: differences of the running sum are exact
    total = torch.zeros(col.numel() + 1, dtype=torch.float64, device="cuda")
    torch.cumsum(val.double() * x[col].double(), 0, out=total[1:])
    want = total[rp[1:]] - total[rp[:-1]]
    torch.cuda.synchronize()
    return rp.to(torch.int32), col.to(torch.int32), val, x, want.to(dtype)


def _us(p, x, y):
    for _ in range(5):
        p.run(x, y)
    ts = []
    for _ in range(7):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            p.run(x, y)
        b.record()
        torch.cuda.synchronize()
        ts.append(a.elapsed_time(b) * 100.0)
    return sorted(ts)[3]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("long_lds", [0, 1, 2, 3])
@pytest.mark.parametrize("longest", [8192, 8193, 60_000])
def test_results(longest, long_lds, dtype):
    n = 700_000
    rp, col, val, x, want = _matrix(5000, n, 6, {17: longest, 18: 1500, 4999: 2000}, dtype)
    p = G.Plan(rp, col, val, n=n, selector="csr_panel",
               params={"long_lds": long_lds} if long_lds else None)
    y = torch.full((5000,), float("nan"), dtype=dtype, device="cuda")
    assert torch.equal(p.run(x, y), want)
    i = p.info()
    # asked for without tiles: the rows above 8192 leave the two-step form
    if long_lds == 2:
        assert i["params"]["panel_xcd"] == (1 if longest > 8192 else 0)
    q = G.Plan(rp, col, val, n=n, selector="csr_panel", params=i["params"])
    assert q.info()["params"] == i["params"] and torch.equal(q.run(x), want)
    r2, c2, v2 = p.roundtrip()
    assert torch.equal(r2, rp) and torch.equal(c2, col) and torch.equal(v2, val)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_no_slower_than_the_xcd_panels(dtype):
    """One row of 900k entries: a workgroup of its own took ten times as long
    as the XCD panels (530 us for 53)."""
    rp, col, val, x, want = _matrix(100_000, 2_000_000, 5, {50_000: 900_000}, dtype)
    y = torch.empty_like(want)
    t = {}
    for name, params in (("default", None), ("no tiles", {"long_lds": 2}),
                         ("xcd", {"panel_xcd": 1})):
        print(name, flush=True)
        p = G.Plan(rp, col, val, n=2_000_000, selector="csr_panel", params=params)
        assert torch.equal(p.run(x, y), want)
        t[name] = _us(p, x, y)
    print(t, flush=True)
    assert t["default"] <= 1.25 * t["xcd"] and t["no tiles"] <= 1.25 * t["xcd"]
