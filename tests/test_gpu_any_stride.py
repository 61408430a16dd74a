"""SpMM with 16-byte accesses at any element-aligned address (the last lane of
a row overlaps its neighbour) and products without a plan, whose long rows are
left to the whole workgroup (csrc/product_impl.hpp).  Exact inputs, so every
result is the oracle's bit for bit, whatever the order of the additions."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import spgen
from _cases import int_valued, matrix, to_gpu

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


# around the vector (2 FP64, 4 FP32), one past each power of two of lanes, more than one slab of columns
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 9, 13, 33, 64, 65, 127, 129, 131])
@pytest.mark.parametrize("vname", ["float64", "float32", "bfloat16"])
@pytest.mark.parametrize("kind", ["empty_rows", "one_long_row", "wide"])
def test_spmm_any_stride_exact(spx, torch, kind, vname, k):
    A = int_valued(matrix(kind, 61))
    vt = getattr(torch, vname)
    xt = torch.float64 if vname == "float64" else torch.float32
    G = to_gpu(A, vt)
    Xh = spgen.small_ints(A.n * k, 62).reshape(A.n, k)
    ref = oracle.spmm(A, Xh)
    assert np.abs(ref).max() < 2 ** 24
    for pad, first in ((0, 0), (1, 1), (3, 2)):  # row strides and first elements off the 16-byte grid
        buf = torch.zeros(A.n * (k + pad) + first, dtype=xt, device="cuda:0")
        X = buf[first:].view(A.n, k + pad)[:, :k]
        X.copy_(torch.from_numpy(Xh))
        out = torch.full((A.m * (k + pad) + first,), 7.0, dtype=xt, device="cuda:0")
        Y = out[first:].view(A.m, k + pad)
        for plan in (None, spx.Plan.for_matrix(G, k=k)):
            out.fill_(7.0)
            spx.spmm(G, X, Y[:, :k], plan=plan)
            got = Y.double().cpu().numpy()
            assert np.array_equal(got[:, :k], ref), (pad, first, plan)
            assert (got[:, k:] == 7.0).all() and (out[:first] == 7.0).all()


@pytest.mark.parametrize("vname", ["float64", "float32", "bfloat16"])
@pytest.mark.parametrize("kind", ["powerlaw", "one_long_row", "wide", "stencil5"])
def test_unplanned_spmv_exact(spx, torch, kind, vname):
    A = int_valued(matrix(kind, 63))
    G = to_gpu(A, getattr(torch, vname))
    xt = torch.float64 if vname == "float64" else torch.float32
    xh = spgen.small_ints(A.n, 64)
    x = torch.from_numpy(xh).to("cuda:0").to(xt)
    ref = oracle.spmv(A, xh)
    assert np.array_equal(spx.spmv(G, x).double().cpu().numpy(), ref)
    y, xs = spx.spmv_save(G, x)
    assert np.array_equal(y.double().cpu().numpy(), ref)
    assert np.array_equal(xs.double().cpu().numpy(), xh[A.colind])
    idx = spx.transpose_index(G)
    dy = spgen.small_ints(A.m, 65)
    got = spx.spmv_t(G, torch.from_numpy(dy).to("cuda:0").to(xt), index=idx)
    assert np.array_equal(got.double().cpu().numpy(), oracle.spmv_t(A, dy))
