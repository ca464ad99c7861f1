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
