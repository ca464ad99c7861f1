"""The binding's two ways to the library: plain calls through csrc/host_call.cpp give what the ctypes calls give, bit for bit, and all other calls
are left to these."""
import pytest
import torch

import paper_1710_08717_amd as la
from paper_1710_08717_amd import binding


def spd(batch, n, dt):
    X = torch.randn(batch, n, n, dtype=dt)
    return X @ X.mT + n * torch.eye(n, dtype=dt)


def calls(L, A, R, y):
    B = la.potri(L)
    return {
        "potrf": lambda: la.potrf(A), "potrf_u": lambda: la.potrf(A, lower=False), "potrf_b": lambda: la.potrf_backward(L, A),
        "trsm": lambda: la.trsm(L, R), "trsm_t": lambda: la.trsm(L, R, trans=True, alpha=0.5), "trsm_r": lambda: la.trsm(L, R.mT.contiguous(), rightside=True),
        "trmm": lambda: la.trmm(L, R), "trsm_b": lambda: la.trsm_backward(L, R, R), "trmm_b": lambda: la.trmm_backward(L, R, R, trans=True),
        "syrk": lambda: la.syrk(R), "syrk_t": lambda: la.syrk(R, trans=True, alpha=2.0), "syrk_b": lambda: la.syrk_backward(R, A),
        "gemm2": lambda: la.gemm2(R, A, ta=True), "gemm2_b": lambda: la.gemm2_backward(R, A, R.mT.contiguous(), ta=True),
        "potri": lambda: la.potri(L), "potri_b": lambda: la.potri_backward(L, B, A), "logdet": lambda: la.sumlogdiag(L),
        "gp": lambda: la.gp_criterion(A, y),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("lead,n,m", [((), 5, 3), ((0,), 4, 2), ((2, 3), 33, 7), ((2,), 300, 20)])
def test_both_ways_agree(dt, lead, n, m, monkeypatch):
    torch.manual_seed(n)
    b = 1
    for s in lead:
        b *= s
    A = spd(b, n, dt).reshape(*lead, n, n).cuda()
    R, y = torch.randn(*lead, n, m, dtype=dt).cuda(), torch.randn(*lead, n, dtype=dt).cuda()
    L = la.potrf(A)
    fast = {k: f() for k, f in calls(L, A, R, y).items()}
    monkeypatch.setattr(binding, "_host", None)
    for k, f in calls(L, A, R, y).items():
        for x, z in zip(*[(t if isinstance(t, tuple) else (t,)) for t in (fast[k], f())]):
            assert x.shape == z.shape and x.dtype == z.dtype and x.device == z.device and not x.requires_grad, k
            assert torch.equal(x, z), k


@pytest.mark.gpu
def test_other_calls_are_left_to_ctypes():
    host = la.load() and binding._host
    A = spd(2, 6, torch.float64).cuda()
    assert host.potrf(A, True) is not None
    for bad in ((A.mT, True), (A.half(), True), (A[:, :5], True), (A.cpu(), True), (A, 1), (A.tolist(), True), (A,),
                (A.to_sparse(), True)):
        assert host.potrf(*bad) is None
    assert host.tri(True, A, A.float(), True, False, False, 1.0) is None
    assert host.tri(True, A, A[:1], True, False, False, 1.0) is None
    assert host.tri(True, A, A, True, False, False, 1) is None
    assert host.gemm2(A, A[:, :5].contiguous(), False, False, 1.0) is None
    from torch.overrides import TorchFunctionMode

    with TorchFunctionMode():
        assert host.potrf(A, True) is None
    seen = []
    torch.func.vmap(lambda x: seen.append(host.potrf(x, True)) or x)(A)
    assert seen == [None]
    for fn in (lambda: la.potrf(A.mT), lambda: la.potrf(A.half()), lambda: la.trsm(A, A.float()), lambda: la.gemm2(A, A.cpu())):
        with pytest.raises(la.LaError):
            fn()
    with pytest.raises(AssertionError):
        la.trsm(A, A[:1].contiguous())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        L = la.potrf(A)
    s.synchronize()
    assert torch.equal(L, la.potrf(A))


def test_host_call_leaves_cpu_tensors():
    la.load()
    A = torch.eye(3)[None]
    assert binding._host.potrf(A, True) is None and binding._host.gp_criterion(A, A[:, 0]) is None
    with pytest.raises(la.LaError):
        la.potrf(A)
