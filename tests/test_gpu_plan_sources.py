"""Plans from CSR arrays at every alignment, read in place or copied first.

The oracle is the float64 product; a row of k entries summed in any order in
the matrix's own type differs from it by at most (k + 2) eps sum |a x|.
"""
import numpy as np
import pytest
import torch

from paper_1210_2536_amd import capi as C
from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


def _shifted(t, shift):
    """A copy of t that starts `shift` values into its storage."""
    buf = torch.empty(t.numel() + shift, dtype=t.dtype, device="cuda")
    buf[shift:] = t.cuda()
    return buf[shift:]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kernel", ["csr_vector", "csr_adaptive", "csr_panel", "coo", "ell",
                                    "bcsr"])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_arrays_may_change_after_the_plan(kernel, dtype, shift):
    rng = np.random.default_rng(3)
    m, n, k = 1031, 1500, 7
    col = np.sort(np.stack([rng.choice(n, k, replace=False) for _ in range(m)]), axis=1)
    rp = torch.arange(0, m * k + 1, k, dtype=torch.int32)
    ci = torch.from_numpy(col.reshape(-1).astype(np.int32))
    va = torch.from_numpy(rng.standard_normal(m * k)).to(dtype)
    x = torch.from_numpy(rng.standard_normal(n)).to(dtype)
    want = (va.double().view(m, k) * x.double()[ci.long()].view(m, k))
    bound = (k + 2) * torch.finfo(dtype).eps * want.abs().sum(1)
    d = [_shifted(t, shift) for t in (rp, ci, va)]
    p = G.Plan(*d, n=n, selector=kernel)
    for t in d:   # the plan keeps nothing of the caller's arrays
        t.fill_(1)
    y = p.run(x.cuda())
    assert p.info()["kernel"] == C.KERNELS.index(kernel)
    err = (y.cpu().double() - want.sum(1)).abs()
    assert bool((err <= bound).all())
    s = torch.cuda.Stream()   # an explicit stream
    s.wait_stream(torch.cuda.current_stream())
    y2 = p.run(x.cuda(), stream=s)
    s.synchronize()
    assert torch.equal(y, y2)
    with pytest.raises(TypeError):
        p.run(x)
