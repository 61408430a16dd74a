"""Patterns with long runs of empty rows: the CSC index and the permutation find
each nonzero's row by walking a tile's rows, or, where a tile (4,096 nonzeros)
spans more than 16,384 rows, by a search per nonzero.  Bit for bit against
numpy, on both sides of that line."""
import numpy as np
import pytest

import spgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def spx():
    import paper_1302_1078_amd as m
    return m


def build(spx, torch, m, n, rows, seed):
    """CSR with one nonzero per entry of `rows` (ascending), columns ascending inside a row."""
    rng = np.random.Generator(np.random.PCG64(seed))
    r = np.asarray(rows, np.int64)
    c = rng.integers(0, n, r.size)
    keys = np.unique(r * n + c)
    r, c = keys // n, (keys % n).astype(np.int32)
    v = spgen.uniform(r.size, seed)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))]).astype(np.int32)
    A = spx.CSR(*(torch.from_numpy(a).to("cuda:0") for a in (rowptr, c, v)), (m, n))
    return A, r, c, v


SPAN = 16_384
CASES = {
    # a tile's first and last nonzero just under, at and over the span apart
    "span-1": (40_000, np.r_[5, 5 + SPAN - 1]),
    "span": (40_000, np.r_[5, 5 + SPAN]),
    "span+1": (40_000, np.r_[5, 5 + SPAN + 1]),
    "first and last row": (3_000_000, np.r_[0, 2_999_999]),
    "one nonzero": (3_000_000, np.r_[1_234_567]),
    "rows of many": (1_000_000, np.repeat([3, 499_999, 999_998], 3000)),
    # the second tile spans a gap, the first and third do not
    "gap in a tile": (1_000_000, np.r_[np.arange(6000), 900_000 + np.arange(6000)]),
    "spread": (2_000_000, np.arange(0, 2_000_000, 397)),
    "rows before and after": (500_000, np.r_[200_000:200_100, 300_000:300_100]),
}


@pytest.mark.parametrize("name", CASES)
def test_index_and_permutation(spx, torch, name):
    m, rows = CASES[name]
    A, r, c, v = build(spx, torch, m, m, rows, len(name))
    idx = spx.transpose_index(A)
    order = np.argsort(c, kind="stable")
    assert np.array_equal(idx.perm.cpu().numpy(), order)
    assert np.array_equal(idx.rowind.cpu().numpy(), r[order])
    assert np.array_equal(idx.colptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(c, minlength=m))]))
    perm = np.random.Generator(np.random.PCG64(7)).permutation(m).astype(np.int32)
    B = spx.permute(A, torch.from_numpy(perm).to("cuda:0"))
    label = np.empty(m, np.int64)
    label[perm] = np.arange(m)
    keys = label[r] * m + label[c]
    order = np.argsort(keys)
    assert np.array_equal(B.colind.cpu().numpy(), keys[order] % m)
    assert np.array_equal(B.values.cpu().numpy(), v[order])
    assert np.array_equal(B.rowptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(keys // m, minlength=m))]))


def best_ms(torch, f):
    times = []
    for _ in range(8):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        torch.cuda.synchronize()
        a.record()
        f()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b))
    return min(times)


def test_time_does_not_follow_the_empty_rows(spx, torch):
    """5,000 nonzeros: the index over 10 M rows (and one column) takes at most 10 times the index over 5,000 rows.
    Walking the rows took 400 times as long, a search 24 dependent loads more."""
    def best(m):
        A, *_ = build(spx, torch, m, 1, np.unique(np.linspace(0, m - 1, 5000).astype(np.int64)), 3)
        return best_ms(torch, lambda: spx.transpose_index(A))
    assert best(10_000_000) <= 10 * best(5_000)


def test_assembly_time_with_many_empty_rows(spx, torch):
    """5,000 triplets of 10 M rows: at most 10 times the assembly of 5,000 rows (rowptr is 40 MB, some 10 us of
    stores; one lane after the other storing each head's 2,000 entries took 50 times as long)."""
    def best(m):
        r = torch.linspace(0, m - 1, 5000, device="cuda:0").to(torch.int32)
        v = torch.ones(5000, dtype=torch.float64, device="cuda:0")
        return best_ms(torch, lambda: spx.from_coo(m, m, r, r, v))
    assert best(10_000_000) <= 10 * best(5_000)


# runs of empty rows before the first, between and after the last triplet, each around the eight rows
# that a lane stores by itself
@pytest.mark.parametrize("gap", [0, 1, 7, 8, 9, 64, 65, 5000])
def test_assembly_row_offsets(spx, torch, gap):
    m = 3 * gap + 130 * (gap + 1) + 1
    r = np.concatenate([[gap, gap], 2 * gap + (gap + 1) * np.arange(130), [m - 1 - gap]]).astype(np.int32)
    c = np.arange(r.size, dtype=np.int32)[::-1].copy()
    v = spgen.uniform(r.size, gap)
    order = np.random.Generator(np.random.PCG64(gap)).permutation(r.size)
    A = spx.from_coo(m, r.size, *(torch.from_numpy(a[order].copy()).to("cuda:0") for a in (r, c, v)))
    want = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))])
    assert np.array_equal(A.rowptr.cpu().numpy(), want)
    assert A.nnz == r.size
