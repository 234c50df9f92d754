"""DIA values from HBM: 4 diagonals at a time, y stored past the caches.

Diagonal counts with every remainder of 4, offsets whose first and last tiles
miss rows or columns, and rectangular matrices.  The oracle is the float64 sum
over the diagonals; D products and sums in double, rounded once, differ from
it by at most (D + 1) eps64 sum |a x| + eps sum |a x|.
"""
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("offs,dn", [((-700, -1, 0, 1, 4099), 0), ((-2, -1, 0, 1, 2, 3), 77),
                                     ((-99991, -2, 0, 1, 3, 513, 1025), -1027),
                                     ((-3, -2, -1, 0, 1, 2, 3, 1000003), 1000)])
def test_groups_of_diagonals(dtype, offs, dn):
    D = len(offs)
    elt = 4 if dtype == torch.float32 else 8
    m = (120 << 20) // (D * elt) + 12345    # just above the line
    n = m + dn
    gen = torch.Generator(device="cuda").manual_seed(D)
    i = torch.arange(m, device="cuda", dtype=torch.int32)
    o = torch.tensor(offs, device="cuda", dtype=torch.int32)
    j = i[:, None] + o
    ok = (j >= 0) & (j < n)
    rp = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    rp[1:] = ok.sum(1).cumsum(0)
    a = torch.randn(m, D, generator=gen, device="cuda", dtype=dtype)
    x = torch.randn(n, generator=gen, device="cuda", dtype=dtype)
    p = G.Plan(rp, j[ok], a[ok], n=n, selector="dia_direct")
    info = p.info()
    assert info["dia_ndiags"] * info["m_pad"] * elt > 120 << 20
    buf = torch.full((m + 3,), 7.0, dtype=dtype, device="cuda")
    y = p.run(x, buf[1:m + 1])              # y off 16-byte boundaries
    assert bool((buf[0] == 7) & (buf[m + 1:] == 7).all())
    want = torch.zeros(m, dtype=torch.float64, device="cuda")
    size = torch.zeros(m, dtype=torch.float64, device="cuda")
    for d in range(D):
        t = a[:, d].double() * x.double()[j[:, d].clamp(0, n - 1).long()]
        t = torch.where(ok[:, d], t, 0.0)
        want += t
        size += t.abs()
    eps = torch.finfo(dtype).eps
    bound = ((D + 1) * torch.finfo(torch.float64).eps + eps) * size
    assert bool(((y.double() - want).abs() <= bound).all())
