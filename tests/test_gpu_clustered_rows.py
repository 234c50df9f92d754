"""Long rows whose columns lie in a band: tiles that hold no entry of their row
block are skipped, and the row blocks are cut for the panels that a band
reaches.  Whole-number data, so results are compared bit for bit."""
import numpy as np
import pytest

from oracle import spmv as O

pytestmark = pytest.mark.gpu


def _band(rng, m, k, window):
    """m rows of k distinct ascending columns within `window` of the diagonal."""
    start = np.clip(np.arange(m) - window // 2, 0, m - window)
    col = start[:, None] + np.sort(rng.permuted(np.tile(np.arange(window), (m, 1)), axis=1)[:, :k],
                                   axis=1)
    return np.arange(0, m * k + 1, k), col.reshape(-1).astype(np.int32)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("kernel", ["csr_adaptive", "csr_panel"])
@pytest.mark.parametrize("x_inf", [False, True], ids=["finite", "inf"])
def test_band_results(kernel, dtype, x_inf):
    import torch
    from paper_1210_2536_amd.spmv import Plan
    rng = np.random.default_rng(81)
    m = 45_000                                     # 3 panels of x in float32, 5 in float64
    rp, col = _band(rng, 3000, 400, 1200)
    col = col + np.repeat(np.arange(3000) * 14, 400).astype(np.int32)   # spread over all panels
    n = m
    val = rng.integers(-4, 5, size=col.size).astype(dtype)
    x = rng.integers(-8, 9, size=n).astype(dtype)
    if x_inf:
        x[20_000] = np.inf
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    p = Plan(t(rp.astype(np.int32)), t(col), t(val), n=n, selector=kernel,
             params={"long_lds": 3, "tile_row_min": 256})
    assert p.info()["params"]["long_lds"] == 3 and p.info()["long_rows"] == 3000
    ok = np.isfinite(x)
    ref, _ = O.spmv_accurate(rp, col, val.astype(np.float64),
                             np.where(ok, x, 0).astype(np.float64))
    bad = np.zeros(3000, dtype=bool)
    bad[np.repeat(np.arange(3000), 400)[~ok[col]]] = True
    y = torch.full((3000,), float("nan"), dtype=t(x).dtype, device="cuda")
    for _ in range(3):      # the skipped tiles' partials stay zero from run to run
        y.fill_(float("nan"))
        got = p.run(t(x), y).cpu().numpy()
        assert np.array_equal(got[~bad], ref[~bad].astype(dtype))
        assert not np.isfinite(got[bad]).any()


def _us(p, x, y):
    import torch
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


def _wide_band(m, k, window, dtype):
    """The same on the GPU, one column drawn from each of k steps of the window."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(82)
    start = (torch.arange(m, device="cuda") - window // 2).clamp(0, m - window)
    step = torch.arange(k, device="cuda") * (window // k)
    col = start[:, None] + step + torch.randint(0, window // k, (m, k), device="cuda", generator=g)
    rp = torch.arange(0, m * k + 1, k, dtype=torch.int32, device="cuda")
    val = torch.rand(m * k, device="cuda", generator=g, dtype=torch.float64).to(dtype)
    return rp, col.reshape(-1).to(torch.int32), val


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("m,k,window", [(100_000, 300, 900), (100_000, 600, 3000)])
def test_band_is_no_slower_than_the_binned_launch(m, k, window, dtype):
    """Defaults against the binned launch (long_lds 2), which took 0.35 to 0.7
    of the time of tiles cut for all panels; a quarter is left for the spread
    of the two measurements."""
    import torch
    from paper_1210_2536_amd.spmv import Plan
    dt = getattr(torch, dtype)
    rp, col, val = _wide_band(m, k, window, dt)
    x = torch.rand(m, device="cuda", dtype=torch.float64).to(dt)
    y = torch.empty(m, dtype=dt, device="cuda")
    binned = Plan(rp, col, val, n=m, selector="csr_adaptive", params={"long_lds": 2})
    default = Plan(rp, col, val, n=m, selector="csr_adaptive")
    tb, td = _us(binned, x, y), _us(default, x, y)
    print(f"binned {tb:.1f} us, default {td:.1f} us", flush=True)
    assert td <= 1.25 * tb
