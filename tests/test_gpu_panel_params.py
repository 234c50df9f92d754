"""Parameters that two-step column panels record: the thresholds in effect."""
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


def _matrix(m, n, k, long_rows, dtype):
    length = torch.full((m,), k, dtype=torch.int64, device="cuda")
    for r, w in long_rows.items():
        length[r] = w
    rp = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=rp[1:])
    row = torch.repeat_interleave(length)
    pos = torch.arange(int(rp[-1]), device="cuda") - rp[row]
    col = pos * (n // length)[row] + row * 5 % (n // length)[row]
    val = (torch.arange(col.numel(), device="cuda") * 7 % 9 - 4).to(dtype)
    return rp.to(torch.int32), col.to(torch.int32), val


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("params,recorded", [
    ({"long_lds": 3, "tile_row_min": 16384, "adaptive_wg_min": 16384}, {"tile_row_min": 4096}),
    ({"long_lds": 3, "tile_row_min": 4096}, {"tile_row_min": 4096}),
    ({"long_lds": 3, "tile_row_min": 1000, "adaptive_wg_min": 500}, {"tile_row_min": 500}),
    ({"long_lds": 2}, {"adaptive_wg_min": 1024}),
    ({"long_lds": 2, "adaptive_wg_min": 300}, {"adaptive_wg_min": 300})])
def test_thresholds_recorded_are_those_in_effect(params, recorded, dtype):
    n = 300_000
    rp, col, val = _matrix(3000, n, 9, {k * 7: 5000 + k for k in range(60)}, dtype)
    x = (torch.arange(n, device="cuda") * 11 % 17 - 8).to(dtype)
    want = G.Plan(rp, col, val, n=n, selector="csr_vector").run(x)
    p = G.Plan(rp, col, val, n=n, selector="csr_panel", params=params)
    i = p.info()
    assert i["params"]["panel_xcd"] == 0 and i["params"]["long_lds"] == params["long_lds"]
    for k, v in recorded.items():
        assert i["params"][k] == v
    assert torch.equal(p.run(x), want)
    q = G.Plan(rp, col, val, n=n, selector="csr_panel", params=i["params"])
    assert q.info()["params"] == i["params"] and q.info()["long_rows"] == i["long_rows"]
    assert torch.equal(q.run(x), want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_tuned_two_step_plan_is_no_slower_than_its_caching_choices(dtype):
    """The search times the two-step form with and without reads past the caches."""
    n = 400_000
    rp, col, val = _matrix(n, n, 20, {}, dtype)
    x = (torch.arange(n, device="cuda") * 11 % 17 - 8).to(dtype)
    y = torch.empty_like(x)
    want = G.Plan(rp, col, val, n=n, selector="csr_vector").run(x)
    p = G.Plan(rp, col, val, n=n, selector="csr_panel", autotune=True)
    assert torch.equal(p.run(x, y), want) and p.info()["tune_rejected"] == 0
    i = p.info()["params"]
    q = G.Plan(rp, col, val, n=n, selector="csr_panel", params=i)
    assert q.info()["params"] == i and torch.equal(q.run(x, y), want)
