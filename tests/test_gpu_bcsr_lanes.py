"""BCSR block rows of every length against the lanes that share them.

A lane takes blocks four at a time, then two, then one, so block rows of 0 to
4 G + 5 blocks (G groups of lanes) meet each remainder; m and n off multiples
of 4 cut the last block row and the last block column.  The oracle is the
float64 product; a row of k stored positions differs from it by at most
(k + 2) eps64 sum |a x| in double sums plus eps of the result's rounding.
"""
import numpy as np
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("lanes", [0, 1, 4, 8, 16, 32, 64])
def test_block_rows_of_every_length(dtype, lanes):
    rng = np.random.default_rng(5)
    most = 4 * max(1, lanes // (4 if dtype == torch.float32 else 8)) + 6
    mb, n = 3 * most, 4 * most + 9
    m = 4 * mb - 3
    rows = []
    for r in range(m):
        k = (r // 4) % most
        bc = np.sort(np.random.default_rng(r // 4).choice(-(-n // 4), k, replace=False))
        c = (bc[:, None] * 4 + np.arange(4)).reshape(-1)
        c = c[c < n]
        rows.append(c[rng.random(c.size) < 0.8])
    rp = np.concatenate([[0], np.cumsum([c.size for c in rows])]).astype(np.int32)
    ci = np.concatenate(rows).astype(np.int32)
    va = torch.from_numpy(rng.standard_normal(ci.size)).to(dtype)
    x = torch.from_numpy(rng.standard_normal(n)).to(dtype)
    t = va.double().numpy() * x.double().numpy()[ci]
    want = np.array([t[rp[r]:rp[r + 1]].sum() for r in range(m)])
    size = np.array([np.abs(t[rp[r]:rp[r + 1]]).sum() for r in range(m)])
    p = G.Plan(torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda(), va.cuda(), n=n,
               selector="bcsr", params={"bcsr_lanes": lanes})
    y = p.run(x.cuda()).double().cpu().numpy()
    eps64 = np.finfo(np.float64).eps
    bound = ((4 * most + 2) * eps64 + torch.finfo(dtype).eps) * size
    assert (np.abs(y - want) <= bound).all()
