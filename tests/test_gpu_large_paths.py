"""Element-by-element parity with the CPU oracle on the code paths only a large single matrix takes
(section 4.2: potrf and its backward expression): potrf right-looking over panels of 2048 columns
(one matrix of n >= 4096), the backward pass as the closed expression with every merge level of the
explicit inverse (n = 2048 in fp32, 2047 in fp64) and as the reverse sweep over the blocked factorisation
by block columns of 1024 (fp64 from n = 2048 on, fp32 at 4096; n = 5376: a ragged last block of 256).  The
tolerances of the operators, relative Frobenius error of the whole matrix."""
import sys
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

TOL = {"f32": 2e-4, "f64": 1e-10}


@pytest.fixture(scope="module")
def la():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_08717_amd as la_mod

    la_mod.load()
    return la_mod


@pytest.fixture(autouse=True)
def _announce(request):
    sys.stderr.write(f"\n[gpu-case] {request.node.nodeid}\n")
    sys.stderr.flush()
    yield


def dev(a):
    import torch

    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch

    torch.cuda.synchronize()
    return t.cpu().numpy()


def relerr(x, ref):
    x = np.asarray(x, dtype=np.float64).ravel()
    ref = np.asarray(ref, dtype=np.float64).ravel()
    return float(np.linalg.norm(x - ref) / np.linalg.norm(ref))


def note(msg):
    sys.stderr.write(f"[large-paths] {msg}\n")
    sys.stderr.flush()


_cache = {}


def problem(n, dtype):
    """One SPD matrix of the C5 recipe at size n (A = X X^T / 2n + I), its oracle factor, Lbar and 512 right-hand sides."""
    key = (n, dtype)
    if key not in _cache:
        _cache.clear()  # one problem at a time: these are big
        w = workloads.make("C5", n=n, m=512, dtype=dtype)
        t = time.time()
        w["L_oracle"] = __import__("oracle").potrf(w["A"])
        note(f"oracle potrf n={n} {dtype}: {time.time() - t:.1f} s")
        _cache[key] = w
    return _cache[key]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_potrf_panel_path_n4096_full_compare(la, orc, dtype):
    w = problem(4096, dtype)
    L = host(la.potrf(dev(w["A"])))
    assert np.all(np.triu(L[0], 1) == 0)
    assert relerr(L, w["L_oracle"]) <= TOL[dtype]
    # the upper factor of the same matrix is the transposed view of the same path
    R = host(la.potrf(dev(w["A"]), lower=False))
    assert np.all(np.tril(R[0], -1) == 0)
    assert relerr(R[0], w["L_oracle"][0].T) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_trsm_block_substitution_n4096_full_compare(la, orc, dtype):
    w = problem(4096, dtype)
    Lr = w["L_oracle"].astype(workloads.np_dtype(dtype))  # the factor as the GPU operator would receive it
    R = w["rhs"]
    for kw in (dict(), dict(trans=True)):
        X = host(la.trsm(dev(Lr), dev(R), **kw))
        assert relerr(X, orc.trsm(Lr, R, **kw)) <= TOL[dtype], kw


@pytest.mark.parametrize("n,dtype", [(2047, "f64"), (2048, "f64"), (2048, "f32")])
def test_backward_closed_expression_n2048_full_compare(la, orc, n, dtype):
    """the largest sizes of the closed expression, and in fp64 the first of the sweep: one matrix of 4 Mi elements"""
    w = problem(n, dtype)
    Lr = w["L_oracle"].astype(workloads.np_dtype(dtype))
    t = time.time()
    ref = orc.potrf_backward(Lr, w["Lbar"])
    note(f"oracle backward n={n} {dtype}: {time.time() - t:.1f} s")
    Abar = host(la.potrf_backward(dev(Lr), dev(w["Lbar"])))
    assert np.array_equal(Abar[0], Abar[0].T)
    assert relerr(Abar, ref) <= TOL[dtype]
    # in place (Abar over Lbar) takes the same path, the closed expression with one more copy
    G = dev(w["Lbar"])
    la.potrf_backward(dev(Lr), G, out=G)
    assert relerr(host(G), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_backward_sweep_n4096_full_compare(la, orc, dtype):
    w = problem(4096, dtype)
    Lr = w["L_oracle"].astype(workloads.np_dtype(dtype))
    t = time.time()
    ref = orc.potrf_backward(Lr, w["Lbar"])
    note(f"oracle backward n=4096 {dtype}: {time.time() - t:.1f} s")
    Abar = host(la.potrf_backward(dev(Lr), dev(w["Lbar"])))
    assert np.array_equal(Abar[0], Abar[0].T)
    assert relerr(Abar, ref) <= TOL[dtype]


def test_potrf_and_backward_sweep_ragged_n5376_full_compare(la, orc):
    """n = 5376 = 2048 + 2048 + 1280: three potrf panels with a ragged last one; the sweep goes by five block columns of
    1024 and a last one of 256."""
    dtype = "f64"
    w = problem(5376, dtype)
    L = host(la.potrf(dev(w["A"])))
    assert relerr(L, w["L_oracle"]) <= TOL[dtype]
    t = time.time()
    ref = orc.potrf_backward(w["L_oracle"], w["Lbar"])
    note(f"oracle backward n=5376 {dtype}: {time.time() - t:.1f} s")
    Abar = host(la.potrf_backward(dev(w["L_oracle"]), dev(w["Lbar"])))
    assert np.array_equal(Abar[0], Abar[0].T)
    assert relerr(Abar, ref) <= TOL[dtype]


@pytest.mark.parametrize("batch,n,dtype,lower", [(1, 10000, "f32", True), (1, 10241, "f64", False), (2, 10000, "f64", True)])
def test_backward_sweep_by_columns_of_two_blocks(la, batch, n, dtype, lower):
    """n >= 10000, up to three matrices: the rule's own expression, multiplied out in 64 bits (the factors have condition numbers of
    about three, so that the errors of Abar are seen at their own size); in place too"""
    import torch

    dt = torch.float64 if dtype == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n)
    L = torch.randn(batch, n, n, generator=g, device="cuda", dtype=dt).tril_().mul_(0.5 / n**0.5)
    L.diagonal(dim1=1, dim2=2).copy_(1 + torch.rand(batch, n, generator=g, device="cuda", dtype=dt))
    G = torch.randn(batch, n, n, generator=g, device="cuda", dtype=dt).tril_()
    if not lower:
        L, G = L.mT.contiguous(), G.mT.contiguous()
    got = la.potrf_backward(L, G, lower=lower)
    inplace = G.clone()
    la.potrf_backward(L, inplace, lower=lower, out=inplace)
    assert torch.equal(inplace, got)
    del inplace
    for b in range(batch):
        assert torch.equal(got[b], got[b].mT)
        F, D = (L[b].double(), G[b].double()) if lower else (L[b].double().mT.contiguous(), G[b].double().mT.contiguous())
        P = (F.mT.contiguous() @ D).tril_()  # 2 L^T Abar L = Phi(L^T Lbar) + its transpose
        P.diagonal().mul_(0.5)
        P = P + P.mT
        assert float((2.0 * (F.mT.contiguous() @ got[b].double() @ F) - P).norm() / P.norm()) <= TOL[dtype]
