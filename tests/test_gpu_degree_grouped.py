"""Degree order from 131,072 nonzeros on, where the columns are first grouped by
their high bits and counted tile by tile in LDS, against numpy: groups of one
column and of more than the LDS window, tiles that span several groups, columns
out of range (not counted), pieces of 2^25 nonzeros."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LINE, PIECE = 1 << 17, 1 << 25


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


def check(torch, n, c):
    import paper_1302_1078_amd as spx
    colind = torch.from_numpy(c).to("cuda:0")
    rowptr = torch.tensor([0, c.size], dtype=torch.int32, device="cuda:0")
    A = spx.CSR(rowptr, colind, torch.empty(0, dtype=torch.float64, device="cuda:0"), (1, n))
    counts = np.bincount(c[(c >= 0) & (c < n)], minlength=n)
    assert np.array_equal(spx.degree_order(A).cpu().numpy(), np.argsort(-counts, kind="stable"))


def draw(n, nnz, kind):
    rng = np.random.Generator(np.random.PCG64(nnz + n))
    c = rng.integers(0, n, nnz)
    if kind == "skewed":
        c = np.minimum((n * rng.random(nnz) ** 6).astype(np.int64), n - 1)
    elif kind == "out_of_range":
        at = rng.random(nnz)
        c = np.where(at < 0.2, -1 - c, np.where(at < 0.4, n + c, c))
        c = np.clip(c, -(1 << 31), (1 << 31) - 1)
    return c.astype(np.int32)


@pytest.mark.parametrize("kind", ["uniform", "skewed", "out_of_range"])
@pytest.mark.parametrize("n", [1, 7, 900, 20_000, 300_000, 5_000_000])
@pytest.mark.parametrize("nnz", [LINE - 1, LINE, 200_000])
def test_degree_order(torch, n, nnz, kind):
    check(torch, n, draw(n, nnz, kind))


@pytest.mark.parametrize("nnz", [PIECE, PIECE + 1, 2 * PIECE + 4097])
def test_degree_order_in_pieces(torch, nnz):
    check(torch, 50_000, draw(50_000, nnz, "skewed"))
