"""Device memory of the two-step column panels: never above the plan's storage
cap, whatever the lengths of the rows the blocks take, and no row pointers kept
twice."""
import numpy as np
import pytest
import torch

from paper_1210_2536_amd import capi as C
from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu

REST = [k for k in C.KERNELS if k != "csr_panel"]


def _matrix(lengths, n, dtype):
    """Rows of the given lengths, columns at even steps from a start of their own."""
    length = torch.from_numpy(np.asarray(lengths)).cuda()
    rp = torch.zeros(length.numel() + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=rp[1:])
    row = torch.repeat_interleave(length)
    pos = torch.arange(int(rp[-1]), device="cuda") - rp[row]
    step = n // length.clamp_min(1)
    start = torch.arange(length.numel(), device="cuda") * 37 % step.clamp_min(1)
    col = pos * step[row] + start[row]
    val = (torch.arange(col.numel(), device="cuda") * 7 % 9 - 4).to(dtype)
    x = (torch.arange(n, device="cuda") * 11 % 17 - 8).to(dtype)
    return rp.to(torch.int32), col.to(torch.int32), val, x


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("kind", ["part_full", "full", "mixed"])
def test_two_steps_stay_inside_the_storage_cap(kind, dtype):
    """One row of 4096 entries sets how far apart blocks start; rows of 2100
    (float64) then leave them half empty, rows of 3100 (float32) a quarter."""
    part = 2100 if dtype == torch.float64 else 3100
    lengths = {"part_full": [part] * 1500 + [4096],
               "full": [60] * 40_000,
               "mixed": [1025, 2047, 4096, 3] * 500 + [9000] * 40}[kind]
    n = 1_200_000
    rp, col, val, x = _matrix(lengths, n, dtype)
    want = G.Plan(rp, col, val, n=n, selector="csr_vector").run(x)
    params = {"tile_row_min": 4096}
    free = G.Plan(rp, col, val, n=n, selector="exhaustive", disable=REST, params=params).info()
    assert free["params"]["panel_xcd"] == 0
    held = free["device_bytes"]
    elt = val.element_size()
    least = col.numel() * (elt + 4) + 16 * (len(lengths) + 1) * (elt + 4)   # the XCD panels'
    forms = set()
    for cap in np.linspace(least, 1.3 * held, 9).astype(np.int64):
        p = G.Plan(rp, col, val, n=n, selector="exhaustive", disable=REST, params=params,
                   mem_cap=int(cap))
        i = p.info()
        assert i["kernel_name"] == "csr_panel"
        if i["params"]["panel_xcd"] == 0 and kind != "mixed":   # (beside a CSR copy there)
            assert i["device_bytes"] <= cap, (int(cap), i["device_bytes"])
        forms.add(i["params"]["panel_xcd"])
        assert torch.equal(p.run(x), want)
    assert forms == {0, 1}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64], ids=["f32", "f64"])
def test_row_pointers_are_held_once(dtype):
    """A row left to another kernel keeps the plan's CSR copy, and with it the
    only row pointers; 400k empty rows make them show."""
    lengths = np.zeros(400_000, dtype=np.int64)
    lengths[::100] = 30
    n = 700_000
    sizes = []
    for longest in (1000, 2000):
        lengths[5] = longest
        rp, col, val, x = _matrix(lengths, n, dtype)
        p = G.Plan(rp, col, val, n=n, selector="csr_panel", params={"long_lds": 2})
        assert p.info()["params"]["panel_xcd"] == 0
        r2, c2, v2 = p.roundtrip()
        assert torch.equal(r2, rp) and torch.equal(c2, col) and torch.equal(v2, val)
        assert torch.equal(p.run(x), G.Plan(rp, col, val, n=n, selector="csr_vector").run(x))
        sizes.append(p.info()["device_bytes"])
    # the longer row adds the copy of columns and values, not of row pointers
    copy = col.numel() * (4 + val.element_size())
    assert sizes[1] - sizes[0] < copy + 400_000 * 4 // 2
