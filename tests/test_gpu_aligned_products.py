"""Products of 16-byte aligned operands, whose slabs go straight from memory to LDS: rows and columns past the end of an operand, last slabs that
are not full, one slab, two and many, each tile size and operand layout, triangles that cross a slab.

Bound: a sum of k products in another order differs from the 64-bit one by at most about k eps |A| |B|; of normal entries that is below
2 sqrt(k) eps of the result's norm (a random walk), held here with a factor of four to spare."""
import numpy as np
import pytest
import torch

import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu


def _eps(dt):
    return torch.finfo(dt).eps


def _rand(rng, dt, *shape):
    return torch.from_numpy(rng.standard_normal(shape)).to("cuda", dt)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,m,n,k", [
    (1, 4, 36, 4), (3, 28, 32, 12), (2, 60, 68, 16), (9, 68, 64, 20), (2, 124, 132, 36), (1, 132, 124, 100),
    (5, 252, 260, 64), (17, 64, 64, 132), (1200, 68, 68, 36), (13, 384, 388, 60), (40, 516, 508, 40), (1, 1028, 1020, 1000), (1, 36, 44, 4100),
])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm2(dt, b, m, n, k, ta, tb):
    rng = np.random.default_rng(b + 7 * m + 11 * n + 13 * k)
    A, B = _rand(rng, dt, b, *((k, m) if ta else (m, k))), _rand(rng, dt, b, *((n, k) if tb else (k, n)))
    C = la.gemm2(A, B, ta=bool(ta), tb=bool(tb)).double()
    a, bb = A.double(), B.double()
    ref = torch.matmul(a.mT.contiguous() if ta else a, bb.mT.contiguous() if tb else bb)
    err = (C - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
    assert float(err.max()) <= 8 * k ** 0.5 * _eps(dt)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n,m", [(132, 36), (260, 132), (512, 128), (1100, 516)])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("trans", [False, True])
def test_trmm_triangles(dt, n, m, lower, trans):
    rng = np.random.default_rng(n + m)
    L = _rand(rng, dt, 2, n, n)
    keep = torch.tril if lower else torch.triu
    X = _rand(rng, dt, 2, n, m)
    T = keep(L.double())
    junk = torch.where(keep(torch.ones_like(L)) > 0, L, torch.full_like(L, float("nan")))
    Y = la.trmm(junk.contiguous(), X, lower=lower, trans=trans).double()
    ref = torch.matmul(T.mT.contiguous() if trans else T, X.double())
    err = (Y - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
    assert float(err.max()) <= 8 * n ** 0.5 * _eps(dt)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,n,k", [(1, 260, 44), (3, 516, 132), (30, 300, 20), (1, 2052, 64)])
def test_syrk_symmetric(dt, b, n, k):
    rng = np.random.default_rng(n + k)
    for trans in (False, True):
        A = _rand(rng, dt, b, *((k, n) if trans else (n, k)))
        C = la.syrk(A, trans=trans)
        assert torch.equal(C, C.mT)
        a = A.double().mT.contiguous() if trans else A.double()
        ref = torch.matmul(a, a.mT.contiguous())
        err = (C.double() - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
        assert float(err.max()) <= 8 * k ** 0.5 * _eps(dt)


@pytest.mark.parametrize("dt,b,n", [(torch.float64, 1, 801), (torch.float64, 2, 1001), (torch.float32, 1, 1026), (torch.float32, 1, 803),
                                    (torch.float64, 3, 333), (torch.float32, 2, 131), (torch.float64, 1, 2501), (torch.float32, 1, 2502),
                                    (torch.float64, 30, 901), (torch.float64, 1, 4099), (torch.float32, 1, 4097)])
@pytest.mark.parametrize("lower", [True, False])
def test_padded_working_copies(dt, b, n, lower):
    """Odd rows: factor and gradient with the whole workspace (working copies with padded rows) and without room for those, on a workspace full of
    NaN: neither a pad nor a triangle that nobody wrote may reach a sum.  Bound: a rounding error is 0.29 eps of its partial sum in the mean, the partial
    sums of n products grow to the result, together 0.17 sqrt(n) eps as a random walk; the factorisation passes that on at most times the square root of
    the matrix's condition number (5), the three sums of the gradient at most times that number: 0.38 and 1.5 of sqrt(n) eps, plus a third."""
    rng = np.random.default_rng(n)
    X = _rand(rng, dt, b, n, n).double()
    A64 = torch.matmul(X, X.mT.contiguous()) / n + torch.eye(n, device="cuda", dtype=torch.float64)
    A = A64.to(dt).contiguous()
    G = _rand(rng, dt, b, n, n)
    lib = la.load()
    code, es = (0, 4) if dt == torch.float32 else (1, 8)
    pad = (n + 16 // es - 1) // (16 // es) * (16 // es)
    ref = torch.linalg.cholesky(A.double().cpu())  # (the reference on the CPU: torch's own solves on the GPU have no memory for the largest of these)
    Gl = (G if lower else G.mT).double().tril().cpu()
    P = torch.matmul(ref.mT, Gl).tril()
    P = P - 0.5 * torch.diag_embed(P.diagonal(dim1=1, dim2=2))
    W = torch.linalg.solve_triangular(ref, torch.linalg.solve_triangular(ref.mT, P, upper=True), upper=False, left=False)
    ref, Ab = ref.cuda(), (0.5 * (W + W.mT)).cuda()
    walk = n ** 0.5 * _eps(dt)
    for short in (0, 1):
        def ws(op):
            full = lib.la_workspace_bytes(op, code, b, n, 0, 0)
            less = short * b * n * pad * es if op == 1 or n >= 800 else 0  # (the factorisation of smaller ones has no such copy)
            return torch.full((max(full - less, full // 2),), 255, dtype=torch.uint8, device="cuda") if full else None
        L = la.potrf(A, lower=lower, workspace=ws(0))
        t = L if lower else L.mT
        assert float(t.triu(1).abs().max()) == 0.0
        assert float(((t.double() - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)).max()) <= 0.5 * walk
        B = la.potrf_backward(L, G, lower=lower, workspace=ws(1))
        assert torch.equal(B, B.mT)
        assert float(((B.double() - Ab).flatten(1).norm(dim=1) / Ab.flatten(1).norm(dim=1)).max()) <= 2 * walk
