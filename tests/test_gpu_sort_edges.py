"""The device sort behind assembly, the CSC index, the value map and the degree
order (csrc/radix.hpp) at the edges of its tiles (4,096 elements), digits
(10 bits a pass) and blocks: everything bit for bit against numpy or the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
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


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def triplets(m, n, nnz, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    r = rng.integers(0, m, nnz).astype(np.int32)
    c = rng.integers(0, n, nnz).astype(np.int32)
    # a third of the entries on one row and column: long runs of one digit, and repeats
    r[::3] = m // 2
    c[::6] = n - 1
    return r, c, spgen.uniform(nnz, seed, spgen.TAG_VALUES)


# one pass of no bits, of 3, of 10; two passes with a width of 6 and of 10; four passes; four with 34 bits
SHAPES = [(1, 1), (3, 2), (1, 1 << 10), (60, 50), (1 << 10, 1 << 10), (70_000, 40_000), (5, (1 << 31) - 1)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("nnz", [1, 63, 4095, 4096, 4097, 33_000])
def test_assembly(spx, torch, shape, nnz):
    m, n = shape
    r, c, v = triplets(m, n, nnz, nnz + m)
    A = spx.from_coo(m, n, dev(torch, r), dev(torch, c), dev(torch, v))
    ref = oracle.csr_from_coo(m, n, r, c, v)
    assert np.array_equal(A.rowptr.cpu().numpy(), ref.rowptr)
    assert np.array_equal(A.colind.cpu().numpy(), ref.colind)
    assert np.array_equal(A.values.cpu().numpy().view(np.uint64), ref.values.view(np.uint64))
    # one index out of range anywhere is reported
    bad = c.copy()
    bad[nnz // 2] = -1
    with pytest.raises(ValueError):
        spx.from_coo(m, n, dev(torch, r), dev(torch, bad), dev(torch, v))


def pattern(m, n, nnz, seed):
    r, c, v = triplets(m, n, nnz, seed)
    keys = np.unique(r.astype(np.int64) * n + c)
    r, c = (keys // n).astype(np.int32), (keys % n).astype(np.int32)
    rowptr = np.zeros(m + 1, np.int32)
    rowptr[1:] = np.cumsum(np.bincount(r, minlength=m))
    return rowptr, r, c


# rows far more than nonzeros (runs of empty rows longer than a tile), and far fewer
@pytest.mark.parametrize("m,n", [(1, 300_000), (3, 900), (200_000, 7), (2_000_000, 1), (30_000, 20_000)])
@pytest.mark.parametrize("nnz", [1, 4096, 4097, 140_000])
def test_csc_index_map_and_degree_order(spx, torch, m, n, nnz):
    rowptr, r, c = pattern(m, n, nnz, nnz + n)
    nnz = c.size
    A = spx.CSR(dev(torch, rowptr), dev(torch, c), dev(torch, spgen.uniform(nnz, 3)), (m, n))
    idx = spx.transpose_index(A)
    perm = np.argsort(c, kind="stable").astype(np.int32)
    counts = np.bincount(c, minlength=n)
    assert np.array_equal(idx.perm.cpu().numpy(), perm)
    assert np.array_equal(idx.rowind.cpu().numpy(), r[perm])
    assert np.array_equal(idx.colptr.cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
    deg = spx.degree_order(A).cpu().numpy()
    assert np.array_equal(deg, np.argsort(-counts, kind="stable"))


# one and two blocks, positions of up to 16, 17 and 23 bits
@pytest.mark.parametrize("nnz", [1, 255, 8191, 8192, 8193, 65_536, 65_537, 70_001, (1 << 22) + 1])
def test_value_map(spx, torch, nnz):
    rng = np.random.Generator(np.random.PCG64(nnz))
    perm = rng.permutation(nnz).astype(np.int32)
    vm = spx.csc_value_map(spx.CSCIndex(None, None, dev(torch, perm)))
    block = 8192
    dest, local = np.empty(nnz, np.int32), np.empty(nnz, np.int32)
    for b in range(0, nnz, block):
        order = np.argsort(perm[b:b + block], kind="stable")
        dest[perm[b:b + block][order]] = b + np.arange(order.size)
        local[b:b + block] = order
    assert np.array_equal(vm.dest.cpu().numpy(), dest)
    assert np.array_equal(vm.local.cpu().numpy().view(np.uint16), local)


@pytest.mark.parametrize("m", [1, 5, 4097, 100_000])
def test_permute_long_and_empty_rows(spx, torch, m):
    rowptr, r, c = pattern(m, m, 3 * m + 9_000, m)
    v = spgen.uniform(c.size, 5)
    A = spx.CSR(dev(torch, rowptr), dev(torch, c), dev(torch, v), (m, m))
    perm = np.random.Generator(np.random.PCG64(m)).permutation(m).astype(np.int32)
    B = spx.permute(A, dev(torch, perm))
    label = np.empty(m, np.int64)
    label[perm] = np.arange(m)
    keys = label[r] * m + label[c]
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(B.colind.cpu().numpy(), keys[order] % m)
    assert np.array_equal(B.values.cpu().numpy(), v[order])
    assert np.array_equal(B.rowptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(keys // m, minlength=m))]))
