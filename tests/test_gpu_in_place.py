"""C calls whose outputs share memory with their inputs: the sort behind them
writes outputs before its last pass, so each buffer order of it (one, two,
three and four passes) is compared with the same call on separate arrays."""
import ctypes

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
def lib(torch):
    from paper_1302_1078_amd import _lib
    return _lib.load()


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def workspace(torch, query, *sizes):
    nb = ctypes.c_size_t()
    assert query(*sizes, ctypes.byref(nb)) == 0
    return torch.empty(max(nb.value, 1), dtype=torch.uint8, device="cuda:0"), nb.value


def stream(torch):
    return torch.cuda.current_stream().cuda_stream


def square(m, nnz, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    keys = np.unique(rng.integers(0, m, nnz) * m + rng.integers(0, m, nnz))
    r, c = (keys // m).astype(np.int32), (keys % m).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=m))]).astype(np.int32)
    return rowptr, r, c, spgen.uniform(c.size, seed)


# 10, 20, 22 and 32 key bits: one, two, three and four passes.  The last has more
# tiles (1,465 of 4,096 nonzeros) than the device holds at once (3 per CU): a
# tile that overwrites another's input is then seen, not only possible.
@pytest.mark.parametrize("m", [30, 1000, 2000, 40_000])
def test_permute_in_place(lib, torch, m):
    rowptr, r, c, v = square(m, {30: 600, 40_000: 6_000_000}.get(m, 300_000), m)
    nnz = c.size
    perm = np.random.Generator(np.random.PCG64(m + 1)).permutation(m).astype(np.int32)
    label = np.empty(m, np.int64)
    label[perm] = np.arange(m)
    keys = label[r] * m + label[c]
    order = np.argsort(keys, kind="stable")
    rp, ci, va, pe = (dev(torch, a) for a in (rowptr, c, v, perm))
    out = torch.empty(1, dtype=torch.int32, device="cuda:0")
    ws, nb = workspace(torch, lib.csr_permute_workspace_bytes, m, nnz)
    assert lib.csr_permute(m, nnz, rp.data_ptr(), ci.data_ptr(), va.data_ptr(), pe.data_ptr(), rp.data_ptr(),
                           ci.data_ptr(), va.data_ptr(), out.data_ptr(), ws.data_ptr(), nb, stream(torch)) == 0
    assert out.item() == nnz
    assert np.array_equal(ci.cpu().numpy(), keys[order] % m)
    assert np.array_equal(va.cpu().numpy(), v[order])
    assert np.array_equal(rp.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(keys // m, minlength=m))]))


@pytest.mark.parametrize("m", [30, 1000, 2000, 40_000])
@pytest.mark.parametrize("over", ["v", "r_and_c"])
def test_assembly_over_its_triplets(lib, torch, m, over):
    nnz = 6_000_000
    rng = np.random.Generator(np.random.PCG64(m))
    r, c = (rng.integers(0, m, nnz).astype(np.int32) for _ in range(2))
    v = spgen.uniform(nnz, m)
    ref = oracle.csr_from_coo(m, m, r, c, v)
    both = dev(torch, np.concatenate([r, c]))  # r and c side by side: as many bytes as v
    tv = dev(torch, v)
    colind = torch.empty(nnz, dtype=torch.int32, device="cuda:0")
    rowptr = torch.empty(m + 1, dtype=torch.int32, device="cuda:0")
    values = tv if over == "v" else both.view(torch.float64)
    out = torch.empty(1, dtype=torch.int32, device="cuda:0")
    ws, nb = workspace(torch, lib.csr_from_coo_workspace_bytes, m, m, nnz)
    assert lib.csr_from_coo(m, m, nnz, both.data_ptr(), both[nnz:].data_ptr(), tv.data_ptr(), rowptr.data_ptr(),
                            colind.data_ptr(), values.data_ptr(), out.data_ptr(), ws.data_ptr(), nb,
                            stream(torch)) == 0
    t = out.item()
    assert t == ref.nnz
    assert np.array_equal(rowptr.cpu().numpy(), ref.rowptr)
    assert np.array_equal(colind[:t].cpu().numpy(), ref.colind)
    assert np.array_equal(values[:t].cpu().numpy().view(np.uint64), ref.values.view(np.uint64))


# 0, 3, 10 and 11 column bits: one pass (which the overlap makes two), and two; 21: three
@pytest.mark.parametrize("n", [1, 7, 1024, 1025, (1 << 20) + 1])
@pytest.mark.parametrize("over", ["rowind", "perm"])
def test_csc_index_over_the_columns(lib, torch, n, over):
    m, nnz = 50_000, 6_000_000
    rng = np.random.Generator(np.random.PCG64(n))
    c = rng.integers(0, n, nnz).astype(np.int32)
    lens = rng.multinomial(nnz, np.full(m, 1.0 / m))
    r = np.repeat(np.arange(m), lens).astype(np.int32)
    rp, ci = dev(torch, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)), dev(torch, c)
    colptr = torch.empty(n + 1, dtype=torch.int32, device="cuda:0")
    other = torch.empty(nnz, dtype=torch.int32, device="cuda:0")
    rowind, perm = (ci, other) if over == "rowind" else (other, ci)
    ws, nb = workspace(torch, lib.csr_transpose_index_workspace_bytes, m, n, nnz)
    assert lib.csr_transpose_index(m, n, nnz, rp.data_ptr(), ci.data_ptr(), colptr.data_ptr(), rowind.data_ptr(),
                                   perm.data_ptr(), ws.data_ptr(), nb, stream(torch)) == 0
    order = np.argsort(c, kind="stable")
    assert np.array_equal(perm.cpu().numpy(), order)
    assert np.array_equal(rowind.cpu().numpy(), r[order])
    assert np.array_equal(colptr.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(c, minlength=n))]))


@pytest.mark.parametrize("nnz", [1, 8192, 9000, 6_000_000])
@pytest.mark.parametrize("over", ["dest", "local"])
def test_value_map_over_perm(lib, torch, nnz, over):
    perm = np.random.Generator(np.random.PCG64(nnz)).permutation(nnz).astype(np.int32)
    ws, nb = workspace(torch, lib.csr_csc_value_map_workspace_bytes, nnz)
    got = {}
    for shared in (False, True):
        p = dev(torch, perm)
        dest = p if shared and over == "dest" else torch.empty(nnz, dtype=torch.int32, device="cuda:0")
        local = p.view(torch.int16)[:nnz] if shared and over == "local" else torch.empty(
            nnz, dtype=torch.int16, device="cuda:0")
        assert lib.csr_csc_value_map(nnz, p.data_ptr(), dest.data_ptr(), local.data_ptr(), ws.data_ptr(), nb,
                                     stream(torch)) == 0
        got[shared] = dest.cpu().numpy(), local.cpu().numpy()
    assert np.array_equal(got[True][0], got[False][0]) and np.array_equal(got[True][1], got[False][1])
