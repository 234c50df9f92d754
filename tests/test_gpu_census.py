"""Diagonal census of matrices whose diagonals overflow its LDS table: exact
counts against the oracle, on both sides of the sizes that choose the bitmap
census, with full, nearly full and short corner diagonals among random ones."""
import numpy as np
import pytest

from oracle import features as OF

pytestmark = pytest.mark.gpu


def _with_diagonals(rng, m, n, per_row, diags):
    """per_row random columns a row plus diagonals (offset, share of its slots)."""
    rows, cols = [np.repeat(np.arange(m), per_row)], [rng.integers(0, n, size=m * per_row)]
    for off, share in diags:
        i = np.arange(max(0, -off), min(m, n - off))
        i = i[rng.random(i.size) < share] if share < 1 else i
        rows.append(i)
        cols.append(i + off)
    key = np.unique(np.concatenate(rows).astype(np.int64) * n + np.concatenate(cols))
    r, c = key // n, (key % n).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))])
    return rp, c


@pytest.mark.parametrize("case", ["square", "wide", "tall", "few_rows", "below_min", "lds_full",
                                  "lds_over", "one_share", "two_parts", "parts_over"])
def test_census_counts(case):
    import torch
    from paper_1210_2536_amd import spmv as G
    rng = np.random.default_rng([76, len(case)])
    m, n, k, diags = {
        "square": (9000, 9000, 20, [(0, 1), (-1, 1), (700, 0.61), (-4000, 0.59), (8990, 1),
                                    (-8999, 1)]),
        "wide": (5000, 40_000, 30, [(0, 1), (20_000, 0.7), (39_999, 1)]),
        "tall": (40_000, 3000, 6, [(0, 1), (-39_000, 0.8), (2999, 1)]),
        "few_rows": (70, 60_000, 2000, [(5, 1), (59_990, 1)]),
        "below_min": (4000, 4000, 30, [(0, 1), (3, 0.65)]),          # under 2^17 entries
        "lds_full": (600_000, 645_185, 3, [(0, 1), (645_180, 1)]),    # 152 KiB of diagonals
        "lds_over": (600_000, 645_186, 3, [(0, 1), (-599_999, 1)]),   # one bit more
        "two_parts": (1_100_000, 1_390_369, 4, [(0, 1), (-1_099_999, 1), (1_390_360, 1)]),
        "parts_over": (1_100_000, 1_390_370, 4, [(0, 1), (1_390_369, 1)]),   # one bit more
        "one_share": (2000, 2000, 66, [(0, 1), (1990, 1)]),
    }[case]
    rp, col = _with_diagonals(rng, m, n, k, diags)
    t = lambda a: torch.from_numpy(a.astype(np.int32)).cuda()  # noqa: E731
    f = G.features(t(rp), t(col), torch.zeros(col.size, device="cuda"), n)
    ref = OF.extract(m, n, rp, col)
    assert ref["ell_feasible"], "no census otherwise"
    for key, name in (("ndiags", "Ndiags"), ("ntdiags", "NTdiags"), ("bandwidth", "bandwidth"),
                      ("max_rd", "max_RD"), ("min_rd", "min_RD"), ("sum_rd", "sum_rd"),
                      ("sum_rd2", "sum_rd2"), ("dia_feasible", "dia_feasible"),
                      ("blocks4", "blocks4")):
        assert int(f[key]) == int(ref[name]), (key, f[key], ref[name])


def test_dia_plan_after_a_bitmap_census():
    """DIA conversion from the bitmap census: over a thousand diagonals, all
    but a few far from full, in a matrix that may still be stored as DIA."""
    import torch
    from paper_1210_2536_amd.spmv import Plan
    rng = np.random.default_rng(77)
    m = 4000
    offs = np.sort(rng.choice(np.arange(-1500, 1501), size=1400, replace=False))
    dense = rng.random((m, offs.size)) < 0.08
    i, j = np.nonzero(dense)
    c = i + offs[j]
    ok = (c >= 0) & (c < m)
    key = np.unique(i[ok].astype(np.int64) * m + c[ok])
    r, col = key // m, (key % m).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))])
    assert col.size > 1 << 17
    val = rng.integers(-4, 5, size=col.size).astype(np.float64)
    x = rng.integers(-8, 9, size=m).astype(np.float64)
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    args = (t(rp.astype(np.int32)), t(col), t(val))
    p = Plan(*args, n=m, selector="dia_direct")
    ref = np.zeros(m)
    np.add.at(ref, r, val * x[col])
    assert np.array_equal(p.run(t(x)).cpu().numpy(), ref)
    for a, b in zip(p.roundtrip(), args):
        assert torch.equal(a, b)
