"""y stored past the caches: DIA with x in LDS and ELL above 120 MB of matrix.

The oracle is the float64 sum over the diagonals; D products and sums in
double, rounded once, differ from it by at most (D + 1) eps64 sum |a x| +
eps sum |a x|.
"""
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kernel,wide", [("dia", 1), ("dia", 2), ("ell", 1), ("ell", 2),
                                         ("dia_direct", 2)])
def test_y_of_large_matrices(dtype, kernel, wide):
    offs, D = (-1025, -3, 0, 1, 2048), 5
    elt = 4 if dtype == torch.float32 else 8
    m = (120 << 20) // (D * elt) + 4321
    gen = torch.Generator(device="cuda").manual_seed(elt)
    j = torch.arange(m, device="cuda", dtype=torch.int32)[:, None] + \
        torch.tensor(offs, device="cuda", dtype=torch.int32)
    ok = (j >= 0) & (j < m)
    rp = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    rp[1:] = ok.sum(1).cumsum(0)
    a = torch.randn(m, D, generator=gen, device="cuda", dtype=dtype)
    x = torch.randn(m, generator=gen, device="cuda", dtype=dtype)
    p = G.Plan(rp, j[ok], a[ok], n=m, selector=kernel,
               params={"wide_loads": wide, "stream_nt": 1})
    buf = torch.full((m + 3,), 7.0, dtype=dtype, device="cuda")
    y = p.run(x, buf[1:m + 1])              # off 16-byte boundaries
    assert bool((buf[0] == 7) & (buf[m + 1:] == 7).all())
    t = torch.where(ok, a.double() * x.double()[j.clamp(0, m - 1).long()], 0.0)
    bound = ((D + 1) * torch.finfo(torch.float64).eps + torch.finfo(dtype).eps) * t.abs().sum(1)
    assert bool(((y.double() - t.sum(1)).abs() <= bound).all())
