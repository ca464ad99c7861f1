"""A few matrices of 16 < n <= 64, one wavefront each: every edge of the two to four tile rows, workgroups of one to four matrices, and sizes
on both sides of the lines where another kernel takes over (256 and 512 matrices, n = 24 of many, vectors of 16, 32, 48, 80 and 128).

Bound: |error| <= 64 n eps of the result's norm; the matrices' condition numbers are about ten, and the forms take a few products with n
terms each (seen: below n eps / 2)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu

NP = {"f64": np.float64, "f32": np.float32}


def close(x, ref, n, dtype):
    x, ref = x.cpu().numpy().astype(np.float64), np.asarray(ref)
    err = np.linalg.norm((x - ref).reshape(len(ref), -1), axis=1) / np.linalg.norm(ref.reshape(len(ref), -1), axis=1)
    return err.max() <= 64 * n * np.finfo(NP[dtype]).eps


def spd(batch, n, seed):
    X = np.random.default_rng(seed).standard_normal((batch, n, 2 * n))
    return np.matmul(X, X.transpose(0, 2, 1)) / (2 * n) + np.eye(n)


def cuda(x, dtype):
    return torch.from_numpy(np.ascontiguousarray(x.astype(NP[dtype]))).cuda()


def junk(x, lower):
    y = x.copy()
    n = x.shape[-1]
    y[:, np.triu(np.ones((n, n), bool), 1) if lower else np.tril(np.ones((n, n), bool), -1)] = np.nan
    return y


def t(x):
    return x.transpose(0, 2, 1)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n", [(1, 17), (5, 18), (3, 24), (2055, 24), (6, 31), (4, 32), (4099, 32), (1026, 25), (1, 33), (257, 47), (257, 48), (7, 48), (2, 49),
                                     (300, 63), (5, 64), (259, 64), (1025, 64)])
def test_factor_operators(batch, n, lower, dtype):
    A = spd(batch, n, n).astype(NP[dtype])
    L = np.linalg.cholesky(A.astype(np.float64))
    F = (L if lower else t(L)).astype(NP[dtype])
    buf = cuda(junk(A, lower), dtype)
    got = la.potrf(buf, lower=lower, out=buf)
    assert close(got, L if lower else t(L), n, dtype)
    assert torch.count_nonzero(got.triu(1) if lower else got.tril(-1)) == 0
    rng = np.random.default_rng(1)
    Fg, F64 = cuda(junk(F, lower), dtype), F.astype(np.float64)
    G, Bbar = (rng.standard_normal((batch, n, n)).astype(NP[dtype]) for _ in range(2))
    Gg = cuda(junk(G, lower), dtype)
    Abar = la.potrf_backward(Fg, Gg, lower=lower)
    assert torch.equal(Abar, Abar.mT)
    assert close(Abar, oracle.potrf_backward(F64, G.astype(np.float64), lower=lower), n, dtype)
    B = la.potri(Fg, lower=lower)
    assert torch.equal(B, B.mT)
    B64 = oracle.potri(F64, lower=lower)
    assert close(B, B64, n, dtype)
    B = B64.astype(NP[dtype])
    X = la.potri_backward(Fg, cuda(B, dtype), cuda(Bbar, dtype), lower=lower)
    assert torch.count_nonzero(X.triu(1) if lower else X.tril(-1)) == 0
    assert close(X, oracle.potri_backward(F64, B.astype(np.float64), Bbar.astype(np.float64), lower=lower), n, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower,trans,rightside", [(True, False, False), (True, True, True), (False, False, True), (False, True, False)])
@pytest.mark.parametrize("batch,n,m", [(1, 17, 1), (5, 23, 16), (3, 24, 7), (4099, 24, 7), (4099, 24, 8), (7, 32, 33), (257, 32, 48), (2, 31, 128), (3, 20, 129), (5, 33, 9), (63, 64, 16), (64, 64, 15),
                                       (6, 44, 32), (6, 45, 33), (4, 60, 16), (4, 61, 16), (5, 49, 49), (2, 64, 80), (3, 44, 128), (257, 47, 48), (257, 64, 128),
                                       (513, 64, 64), (513, 50, 17), (520, 48, 16), (1030, 64, 40)])
def test_products_and_solves(batch, n, m, lower, trans, rightside, dtype):
    L = np.linalg.cholesky(spd(batch, n, 7))
    F = (L if lower else t(L)).astype(NP[dtype])
    rng = np.random.default_rng(2)
    shape = (batch, m, n) if rightside else (batch, n, m)
    X, Xbar = (rng.standard_normal(shape).astype(NP[dtype]) for _ in range(2))
    Fg = cuda(junk(F, lower), dtype)
    M = t(F.astype(np.float64)) if trans else F.astype(np.float64)
    X64, Xb64 = X.astype(np.float64), Xbar.astype(np.float64)
    ref = t(np.linalg.solve(t(M), t(X64))) if rightside else np.linalg.solve(M, X64)
    buf = cuda(X, dtype)
    opt = dict(lower=lower, trans=trans, rightside=rightside)
    assert close(la.trsm(Fg, buf, alpha=-1.5, out=buf, **opt), -1.5 * ref, n, dtype)
    buf = cuda(X, dtype)
    assert close(la.trmm(Fg, buf, alpha=0.5, out=buf, **opt), 0.5 * (X64 @ M if rightside else M @ X64), n, dtype)
    Abar, Lbar = la.trmm_backward(Fg, cuda(X, dtype), cuda(Xbar, dtype), **opt)
    assert close(Abar, Xb64 @ t(M) if rightside else t(M) @ Xb64, n, dtype)
    G = t(X64) @ Xb64 if rightside else Xb64 @ t(X64)
    G = t(G) if trans else G
    assert close(Lbar, np.tril(G) if lower else np.triu(G), n, dtype)
    S = la.syrk(cuda(X, dtype), trans=rightside)
    assert torch.equal(S, S.mT)
    assert close(S, t(X64) @ X64 if rightside else X64 @ t(X64), max(n, m), dtype)
    B = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    B64 = B.astype(np.float64) + t(B.astype(np.float64))
    assert close(la.syrk_backward(cuda(X, dtype), cuda(B, dtype), trans=rightside), X64 @ B64 if rightside else B64 @ X64, n, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("pivot", [0.0, -1.0, float("nan")])
@pytest.mark.parametrize("n", [18, 24, 32, 41, 64])
def test_failing_pivots(n, pivot, dtype):
    """info is the first failing pivot, and the columns before it are right"""
    A = np.repeat(spd(1, n, 5), n + 1, axis=0)
    ref = np.linalg.cholesky(A[-1])
    for k in range(n):
        A[k, k, :] = A[k, :, k] = 0.0
        A[k, k, k] = pivot
    info = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    L = la.potrf(cuda(A, dtype), info=info).cpu().numpy().astype(np.float64)
    assert info.tolist() == list(range(1, n + 1)) + [0]
    for k in range(n):
        want = ref[:, :k].copy()
        want[k] = 0.0
        keep = np.arange(n) != k
        assert np.abs(L[k][keep, :k] - want[keep]).max(initial=0.0) <= 64 * n * np.finfo(NP[dtype]).eps
    assert close(torch.from_numpy(L[-1:]), ref[None], n, dtype)
