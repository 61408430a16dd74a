"""The CSC index of patterns whose column ids are out of range: the call's result
is then unspecified, but it writes nothing outside its output arrays."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 64


@pytest.mark.parametrize("n,cols", [(0, [0]), (0, [5, 0, 3]), (0, list(range(5000))), (1, [0, 7, -1]),
                                    (5, [-3, 4, 12, 0, 2_000_000_000]), (1500, [1499, 1500, -1] * 2000)])
def test_colptr_stays_in_bounds(n, cols):
    torch = pytest.importorskip("torch")
    from paper_1302_1078_amd import _lib
    lib = _lib.load()
    nnz = len(cols)
    buf = torch.full((n + 1 + 2 * GUARD,), -77, dtype=torch.int32, device="cuda:0")
    colptr = buf[GUARD:]
    rowptr = torch.tensor([0, nnz], dtype=torch.int32, device="cuda:0")
    colind = torch.tensor(cols, dtype=torch.int64).to(torch.int32).to("cuda:0")
    rowind, perm = (torch.empty(nnz, dtype=torch.int32, device="cuda:0") for _ in range(2))
    nb = ctypes.c_size_t()
    assert lib.csr_transpose_index_workspace_bytes(1, n, nnz, ctypes.byref(nb)) == 0
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda:0")
    assert lib.csr_transpose_index(1, n, nnz, rowptr.data_ptr(), colind.data_ptr(), colptr.data_ptr(),
                                   rowind.data_ptr(), perm.data_ptr(), ws.data_ptr(), nb.value,
                                   torch.cuda.current_stream().cuda_stream) == 0
    out = buf.cpu().numpy()
    assert (out[:GUARD] == -77).all() and (out[GUARD + n + 1:] == -77).all()
    assert out[GUARD + n] == nnz
    # rowind and perm are whole: every position once, all in row 0
    assert np.array_equal(np.sort(perm.cpu().numpy()), np.arange(nnz))
    assert (rowind.cpu().numpy() == 0).all()
