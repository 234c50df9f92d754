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


def _matrix(short):
    """Rows of LONG entries (columns 0 .. LONG - 1) and, last, one row for each
    length in `short`; every value 1."""
    long_rows = ROWS - len(short)
    nnz = long_rows * LONG + sum(short)
    assert nnz < (1 << 31) - 1
    col = torch.empty(nnz, dtype=torch.int32, device="cuda")
    one = torch.arange(LONG, dtype=torch.int32, device="cuda")
    col[:long_rows * LONG].view(long_rows, LONG).copy_(one)
    at = long_rows * LONG
    ends = [k * LONG for k in range(long_rows + 1)]
    for s in short:
        col[at:at + s] = one[:s]
        at += s
        ends.append(at)
    rp = torch.tensor(ends, dtype=torch.int32, device="cuda")
    return rp, col, torch.ones(nnz, dtype=torch.float32, device="cuda")


def _x_and_sums(short):
    x = (torch.arange(LONG, device="cuda") * 7 % 5 - 1).to(torch.float32)
    want = torch.full((ROWS,), float(x.double().sum()), dtype=torch.float32, device="cuda")
    for k, s in enumerate(short):
        want[ROWS - len(short) + k] = float(x[:s].double().sum())
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
