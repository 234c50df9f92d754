"""Entry positions close to 2^31, the limit of the int32 paths.

Two billion float32 entries in rows of 262272, so that a position moved on by
another row's length would leave the int32 range.  x holds whole numbers whose
row sums are exact in any order.
"""
import pytest
import torch

from paper_1210_2536_amd import spmv as G

pytestmark = pytest.mark.gpu

ROWS, LONG = 8192, 262_272


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch.cuda.empty_cache()


def _matrix(short, short_last=True):
    """Rows of LONG entries (columns 0 .. LONG - 1) and, last or first, one row
    for each length in `short`; every value 1."""
    long_rows = ROWS - len(short)
    lengths = [LONG] * long_rows
    lengths = lengths + short if short_last else short + lengths
    ends = [0]
    for k in lengths:
        ends.append(ends[-1] + k)
    nnz = ends[-1]
    assert nnz < (1 << 31) - 1
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    one = torch.arange(LONG, dtype=torch.int32, device="cuda")
    at = 0 if short_last else sum(short)
    col[at:at + long_rows * LONG].view(long_rows, LONG).copy_(one)
    for k, end in zip(lengths, ends[1:]):
        if k < LONG:
            col[end - k:end] = one[:k]
    rp = torch.tensor(ends, dtype=torch.int32, device="cuda")
    return rp, col, torch.ones(nnz, dtype=torch.float32, device="cuda")


def _x_and_sums(short, short_last=True):
    x = (torch.arange(LONG, device="cuda") * 7 % 5 - 1).to(torch.float32)
    want = torch.full((ROWS,), float(x.double().sum()), dtype=torch.float32, device="cuda")
    for k, s in enumerate(short):
        want[ROWS - len(short) + k if short_last else k] = float(x[:s].double().sum())
    return x, want


def test_batch_rows_of_unequal_length_at_the_last_entries():
    """Two row groups of a batch tile, the second with one entry a row where
    the first has 262272, 508 entries below 2^31."""
    short = [1, 1, 1, 1]
    rp, col, val = _matrix(short)
    x, want = _x_and_sums(short)
    print(f"nnz {col.numel()}", flush=True)
    p = G.Plan(rp, col, val, n=LONG, selector="csr_vector", params={"vector_lanes": 64})
    del col, val
    y = torch.full((ROWS,), -7.0, dtype=torch.float32, device="cuda")
    G.Batch([p]).run([x], [y])
    torch.cuda.synchronize()
    assert torch.equal(y, want)


def test_tiles_of_the_last_rows():
    """Long rows packed into tiles, the last of them ending two entries below
    2^31: the packing lanes step past its end."""
    short = [127, 127, 128, 128]
    rp, col, val = _matrix(short, short_last=False)
    assert col.numel() == (1 << 31) - 2
    x, want = _x_and_sums(short, short_last=False)
    print(f"nnz {col.numel()}", flush=True)
    p = G.Plan(rp, col, val, n=LONG, selector="csr_adaptive")
    assert p.info()["params"]["long_lds"] == 3 and p.info()["long_rows"] == ROWS - 4
    del col, val
    y = torch.full((ROWS,), -7.0, dtype=torch.float32, device="cuda")
    p.run(x, y)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
