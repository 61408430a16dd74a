"""Device memory that the per-pattern calls ask for (the plan keeps its hot-x
workspace as long as it lives)."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def lib():
    from paper_1302_1078_amd import _lib
    return _lib.load()


def query(f, *sizes):
    nb = ctypes.c_size_t()
    assert f(*sizes, ctypes.byref(nb)) == 0
    return nb.value


SLACK = 64 * 256  # array starts are rounded up


@pytest.mark.parametrize("n,nnz", [(1 << 20, 16_800_000), (1 << 19, 10_500_000), (1 << 20, 300_000_000),
                                   (1000, 2_000_000_000)])
@pytest.mark.parametrize("hot", [1024, 65_536])
def test_hot_x(lib, n, nnz, hot):
    """The plan's column indices (4 bytes per nonzero), hot columns and their x, a rank and a slot per column; what
    the ranking needs meanwhile lies over them (and takes up to 5 bytes for each of 2^25 nonzeros)."""
    assert query(lib.csr_plan_hot_x_workspace_bytes, n, nnz, hot) <= 4 * nnz + min(nnz, 1 << 25) + 12 * hot + \
        24 * n + SLACK


def test_degree_order_does_not_grow_with_the_nonzeros(lib):
    n = 1 << 20
    sizes = [query(lib.csr_degree_order_workspace_bytes, n, nnz) for nnz in (50_000_000, 300_000_000, 2_000_000_000)]
    assert max(sizes) <= 21 * n + (5 << 25) + SLACK


@pytest.mark.parametrize("n,per", [(7, 21), (1 << 20, 21), ((1 << 20) + 1, 29), ((1 << 31) - 1, 29)])
def test_csc_index(lib, n, per):
    """Row, two key arrays and a 64-bit payload, and a second payload above two sort passes (20 column bits)."""
    nnz = 10_000_000
    assert query(lib.csr_transpose_index_workspace_bytes, 1000, n, nnz) <= per * nnz + SLACK
