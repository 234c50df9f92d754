"""Batch tiles of two csr_vector row groups, and levels taken from the last.

A level large enough for two row groups a tile, with empty rows, rows longer
and shorter than its lanes and a last tile that is cut, beside a small level:
every row must equal the plan's own run bit for bit, as in any batch.
"""
import numpy as np
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


def _plan(rng, m, n, dtype, lanes):
    length = rng.integers(0, 3 * lanes, size=m)
    length[rng.random(m) < 0.2] = 0
    length[-1] = 2 * lanes + 1
    rp = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    # ascending columns: a start and steps of at least one
    row = np.repeat(np.arange(m), length)
    k = np.arange(rp[-1]) - rp[row]
    col = (row * 7) % (n - 4 * lanes) + k
    val = rng.standard_normal(rp[-1])
    t = lambda a, d: torch.from_numpy(a).to(d).cuda()  # noqa: E731
    return G.Plan(t(rp, torch.int32), t(col.astype(np.int32), torch.int32), t(val, dtype), n=n,
                  selector="csr_vector", params={"vector_lanes": lanes})


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("lanes", [4, 8, 16, 32, 64])
def test_two_row_groups(dtype, lanes):
    rng = np.random.default_rng(lanes)
    per = 256 // lanes
    plans = [_plan(rng, m, m + 500, dtype, lanes)
             for m in (2 * per * 1024 + per + 3, 2 * per * 1024 - 1, 37)]
    xs = [torch.from_numpy(rng.standard_normal(p.n)).to(dtype).cuda() for p in plans]
    ys = [torch.full((p.m,), 7.0, dtype=dtype, device="cuda") for p in plans]
    b = G.Batch(plans)
    b.run(xs, ys)
    for p, x, y in zip(plans, xs, ys):
        assert torch.equal(y, p.run(x))
