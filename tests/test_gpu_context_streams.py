"""A differentiation context built on one stream and used on another."""
import numpy as np
import pytest

import oracle
import spgen
from _cases import matrix, to_gpu

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


@pytest.mark.parametrize("mode", [0, 1])
def test_nothing_is_queued_when_the_constructor_returns(spx, torch, mode):
    """Large enough that whatever the constructor leaves behind is still running: the value map of
    20 M nonzeros takes some hundred microseconds."""
    m, per = 1_000_000, 20
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    rowptr = torch.arange(0, m * per + 1, per, dtype=torch.int32, device="cuda")
    colind = torch.randint(0, m, (m * per,), generator=g, device="cuda", dtype=torch.int32)
    A = spx.CSR(rowptr, colind, torch.ones(m * per, device="cuda"), (m, m))
    for _ in range(3):
        ctx = spx.GradContext(A, mode=mode)
        assert torch.cuda.current_stream().query()
        del ctx


@pytest.mark.parametrize("k", [1, 4])
def test_step_on_another_stream(spx, torch, k):
    A = matrix("powerlaw", seed=3)
    G = to_gpu(A)
    x = spgen.uniform(A.n * k, 4).reshape((A.n, k) if k > 1 else A.n)
    dy = spgen.uniform(A.m * k, 5).reshape((A.m, k) if k > 1 else A.m)
    v = G.values.clone().requires_grad_()
    xt = torch.from_numpy(x).to("cuda").requires_grad_()
    dyt = torch.from_numpy(dy).to("cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx = spx.GradContext(G, k=k)
    with torch.cuda.stream(side):
        y = spx.spmv_autograd(v, xt, ctx)
        dw, dx = torch.autograd.grad(y, (v, xt), dyt)
    side.synchronize()
    cols = [(dy, x)] if k == 1 else [(dy[:, j], x[:, j]) for j in range(k)]
    ref = np.sum([oracle.sddmm(A, np.ascontiguousarray(a), np.ascontiguousarray(b)) for a, b in cols], axis=0)
    assert oracle.rel2(dw.cpu().numpy(), ref) <= 1e-12
    got = dx.cpu().numpy().reshape(A.n, k)
    for j, (a, _) in enumerate(cols):
        assert oracle.rel2(got[:, j], oracle.spmv_t(A, np.ascontiguousarray(a))) <= 1e-12
