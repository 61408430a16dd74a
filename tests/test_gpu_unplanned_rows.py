"""Products without a plan on rows around the line from which a workgroup, not
a row group, serves a row: the line depends on how many long rows a workgroup
has, so blocks of 64 rows hold a given number of them, of lengths on both
sides.  Small integers: every partial sum is exact, whichever way a row goes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def matrix(per_block, other, seed):
    """Blocks of 64 rows, `per_block` of them long (33 to 6,000 nonzeros), the others of up to `other`."""
    rng = np.random.Generator(np.random.PCG64(seed))
    m, n = 64 * 40 + 17, 7000
    lens = rng.integers(0, other + 1, m)
    for b in range(0, m - 64, 64):
        at = b + rng.permutation(64)[:per_block]
        # one length a block, one more or less for some: rows on both sides of whatever line the block has
        base = int(round(np.exp(rng.uniform(np.log(33), np.log(5999)))))
        lens[at] = base + rng.integers(-1, 2, at.size)
    cols = np.concatenate([np.sort(rng.permutation(n)[:l]) for l in lens] + [np.zeros(0, np.int64)]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    values = rng.integers(-3, 4, cols.size).astype(np.float64)
    return oracle.CSR(m, n, rowptr, cols, values)


@pytest.mark.parametrize("per_block", [0, 1, 2, 3, 8, 16, 32, 33, 64])
@pytest.mark.parametrize("other", [1, 12])
@pytest.mark.parametrize("vname,k", [("f64", 1), ("f64", 3), ("f64", 16), ("f32", 1), ("f32", 2), ("f32", 8),
                                     ("bf16", 1), ("bf16", 32)])
def test_exact(torch, per_block, other, vname, k):
    import paper_1302_1078_amd as spx
    A = matrix(per_block, other, 100 * per_block + other)
    vt = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[vname]
    xt = torch.float64 if vname == "f64" else torch.float32
    G = spx.CSR(torch.from_numpy(A.rowptr).cuda(), torch.from_numpy(A.colind).cuda(),
                torch.from_numpy(A.values).to(vt).cuda(), (A.m, A.n))
    X = np.random.Generator(np.random.PCG64(k)).integers(-3, 4, (A.n, k)).astype(np.float64)
    Xt = torch.from_numpy(X).to(xt).cuda()
    if k == 1:
        y = spx.spmv(G, Xt[:, 0].contiguous())
        got = y.cpu().numpy()[:, None]
        ys, xs = spx.spmv_save(G, Xt[:, 0].contiguous())
        assert torch.equal(ys.view(torch.int8), y.view(torch.int8))
        assert np.array_equal(xs.cpu().numpy(), X[A.colind, 0])
    else:
        got = spx.spmm(G, Xt).cpu().numpy()
    for j in range(k):
        assert np.array_equal(got[:, j], oracle.spmv(A, np.ascontiguousarray(X[:, j])))
