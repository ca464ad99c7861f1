"""Many matrices of 32 < n <= 64, one wavefront each: every tile edge of the two sizes of kernel, both triangles with junk in
the other one, in place, failing pivots, vectors of every remainder and a batch that leaves the last workgroup part empty."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 2e-4}
NP = {"f64": np.float64, "f32": np.float32}
BATCH = 1539
SIZES = [33, 37, 47, 48, 49, 63, 64]


def spd(n, seed, dtype):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((BATCH, n, 2 * n))
    return (np.matmul(X, X.transpose(0, 2, 1)) / (2 * n) + np.eye(n)).astype(NP[dtype])


def rel(x, ref):
    x = x.cpu().numpy().astype(np.float64).reshape(x.shape[0], -1)
    ref = np.asarray(ref).reshape(ref.shape[0], -1)
    return np.max(np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1))


def junk(x, lower):
    y = x.copy()
    n = x.shape[-1]
    y[:, np.triu(np.ones((n, n), bool), 1) if lower else np.tril(np.ones((n, n), bool), -1)] = np.nan
    return y


def factor(n, lower, dtype):
    L = np.linalg.cholesky(spd(n, n, "f64"))
    return (L if lower else L.transpose(0, 2, 1).copy()).astype(NP[dtype])


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("n", SIZES)
def test_factor_operators(n, lower, dtype):
    A = spd(n, n, dtype)
    ref = np.linalg.cholesky(A.astype(np.float64))
    buf = torch.from_numpy(junk(A, lower)).cuda()
    L = la.potrf(buf, lower=lower, out=buf)
    assert rel(L, ref if lower else ref.transpose(0, 2, 1)) <= TOL[dtype]
    assert torch.count_nonzero(L.triu(1) if lower else L.tril(-1)) == 0

    rng = np.random.default_rng(1)
    F = factor(n, lower, dtype)
    Fj = torch.from_numpy(junk(F, lower)).cuda()
    Lbar = rng.standard_normal((BATCH, n, n)).astype(NP[dtype])
    Abar = la.potrf_backward(Fj, torch.from_numpy(junk(Lbar, lower)).cuda(), lower=lower)
    assert torch.equal(Abar, Abar.mT)
    assert rel(Abar, oracle.potrf_backward(F.astype(np.float64), Lbar.astype(np.float64), lower=lower)) <= TOL[dtype]

    buf = Fj.clone()
    B = la.potri(buf, lower=lower, out=buf)
    assert torch.equal(B, B.mT)
    Bref = oracle.potri(F.astype(np.float64), lower=lower)
    assert rel(B, Bref) <= TOL[dtype]

    B = Bref.astype(NP[dtype])
    Bbar = rng.standard_normal((BATCH, n, n)).astype(NP[dtype])
    G = la.potri_backward(Fj, torch.from_numpy(B).cuda(), torch.from_numpy(Bbar).cuda(), lower=lower)
    assert torch.count_nonzero(G.triu(1) if lower else G.tril(-1)) == 0
    assert rel(G, oracle.potri_backward(F.astype(np.float64), B.astype(np.float64), Bbar.astype(np.float64), lower=lower)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("rightside", [False, True])
@pytest.mark.parametrize("lower,trans", [(True, False), (True, True), (False, False), (False, True)])
@pytest.mark.parametrize("n,m", [(33, 1), (37, 16), (40, 33), (45, 15), (47, 49), (48, 65), (49, 50), (64, 128)])
def test_solves(n, m, lower, trans, rightside, dtype):
    F = factor(n, lower, dtype)
    rng = np.random.default_rng(2)
    X = rng.standard_normal((BATCH, m, n) if rightside else (BATCH, n, m)).astype(NP[dtype])
    M = np.tril(F) if lower else np.triu(F)
    M = (M.transpose(0, 2, 1) if trans else M).astype(np.float64)
    if rightside:
        ref = np.linalg.solve(M.transpose(0, 2, 1), X.transpose(0, 2, 1).astype(np.float64)).transpose(0, 2, 1)
    else:
        ref = np.linalg.solve(M, X.astype(np.float64))
    buf = torch.from_numpy(X).cuda()
    got = la.trsm(torch.from_numpy(junk(F, lower)).cuda(), buf, lower=lower, trans=trans, rightside=rightside, alpha=-1.5, out=buf)
    assert rel(got, -1.5 * ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [37, 64])
def test_first_failing_pivot(n, dtype):
    A = spd(n, 3, dtype)
    for k in range(n):
        A[k, k, k] = -1.0
    info = torch.zeros(BATCH, dtype=torch.int32, device="cuda")
    la.potrf(torch.from_numpy(A).cuda(), info=info)
    assert info[:n].tolist() == list(range(1, n + 1))
    assert torch.count_nonzero(info[n:]) == 0


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower,trans,rightside", [(True, False, False), (True, True, True), (False, False, True), (False, True, False)])
@pytest.mark.parametrize("n,m", [(33, 1), (37, 16), (48, 17), (49, 33), (63, 48), (64, 65)])
def test_products(n, m, lower, trans, rightside, dtype):
    """trmm (in place), its rule, syrk and its rule, against the definitions in 64 bits"""
    F = factor(n, lower, dtype)
    rng = np.random.default_rng(4)
    shape = (BATCH, m, n) if rightside else (BATCH, n, m)
    X, Xbar = (rng.standard_normal(shape).astype(NP[dtype]) for _ in range(2))
    Fj = torch.from_numpy(junk(F, lower)).cuda()
    M = (np.tril(F) if lower else np.triu(F)).astype(np.float64)
    t = (lambda x: x.transpose(0, 2, 1))
    Mt, X64, Xb64 = (t(M) if trans else M), X.astype(np.float64), Xbar.astype(np.float64)
    buf = torch.from_numpy(X).cuda()
    got = la.trmm(Fj, buf, lower=lower, trans=trans, rightside=rightside, alpha=0.5, out=buf)
    assert rel(got, 0.5 * (X64 @ Mt if rightside else Mt @ X64)) <= TOL[dtype]

    Abar, Lbar = la.trmm_backward(Fj, torch.from_numpy(X).cuda(), torch.from_numpy(Xbar).cuda(), lower=lower, trans=trans,
                                  rightside=rightside)
    assert rel(Abar, Xb64 @ t(Mt) if rightside else t(Mt) @ Xb64) <= TOL[dtype]
    G = t(X64) @ Xb64 if rightside else Xb64 @ t(X64)  # gradient of t(M)
    G = t(G) if trans else G
    assert rel(Lbar, np.tril(G) if lower else np.triu(G)) <= TOL[dtype]
    assert torch.count_nonzero(Lbar.triu(1) if lower else Lbar.tril(-1)) == 0

    S = la.syrk(torch.from_numpy(X).cuda(), trans=rightside, alpha=-2.0)  # n x n from n x m, or from m x n transposed
    assert torch.equal(S, S.mT)
    assert rel(S, -2.0 * (t(X64) @ X64 if rightside else X64 @ t(X64))) <= TOL[dtype]
    B = rng.standard_normal((BATCH, n, n)).astype(NP[dtype])
    B64 = B.astype(np.float64) + t(B.astype(np.float64))
    got = la.syrk_backward(torch.from_numpy(X).cuda(), torch.from_numpy(B).cuda(), trans=rightside)
    assert rel(got, X64 @ B64 if rightside else B64 @ X64) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n,m", [(1, 33, 49), (5, 48, 65), (6, 49, 300), (3, 64, 64)])
def test_few_matrices_without_a_workspace(batch, n, m, lower, dtype):
    """the operators that take scratch for small batches of these sizes, on none"""
    rng = np.random.default_rng(6)
    F = factor(n, lower, dtype)[:batch]
    X, Xbar = (rng.standard_normal((batch, n, m)).astype(NP[dtype]) for _ in range(2))
    Bbar = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    M = (np.tril(F) if lower else np.triu(F)).astype(np.float64)
    t = (lambda x: x.transpose(0, 2, 1))
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    Fj = torch.from_numpy(junk(F, lower)).cuda()
    Xg, Xbg = torch.from_numpy(X).cuda(), torch.from_numpy(Xbar).cuda()
    ref = np.linalg.solve(M, X.astype(np.float64))
    assert rel(la.trsm(Fj, Xg, lower=lower, workspace=none), ref) <= TOL[dtype]
    assert rel(la.trmm(Fj, Xg, lower=lower, workspace=none), M @ X.astype(np.float64)) <= TOL[dtype]
    buf = Xg.clone()
    assert rel(la.trmm(Fj, buf, lower=lower, trans=True, out=buf, workspace=none), t(M) @ X.astype(np.float64)) <= TOL[dtype]
    Y, Lbar = la.trsm_backward(Fj, torch.from_numpy(ref.astype(NP[dtype])).cuda(), Xbg, lower=lower, workspace=none)
    Yref = np.linalg.solve(t(M), Xbar.astype(np.float64))
    assert rel(Y, Yref) <= TOL[dtype]
    G = -Yref @ t(ref)
    assert rel(Lbar, np.tril(G) if lower else np.triu(G)) <= TOL[dtype]
    B = oracle.potri(F.astype(np.float64), lower=lower).astype(NP[dtype])
    got = la.potri_backward(Fj, torch.from_numpy(B).cuda(), torch.from_numpy(Bbar).cuda(), lower=lower, workspace=none)
    assert rel(got, oracle.potri_backward(F.astype(np.float64), B.astype(np.float64), Bbar.astype(np.float64), lower=lower)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n,m", [(1, 17, 129), (5, 24, 200), (6, 31, 700), (3, 32, 130)])
def test_few_solves_of_17_to_32_rows_without_a_workspace(batch, n, m, lower, dtype):
    rng = np.random.default_rng(7)
    F = factor(n, lower, dtype)[:batch]
    X, Xbar = (rng.standard_normal((batch, n, m)).astype(NP[dtype]) for _ in range(2))
    M = (np.tril(F) if lower else np.triu(F)).astype(np.float64)
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    Fj, buf = torch.from_numpy(junk(F, lower)).cuda(), torch.from_numpy(X).cuda()
    ref = np.linalg.solve(M, X.astype(np.float64))
    assert rel(la.trsm(Fj, buf, lower=lower, workspace=none), ref) <= TOL[dtype]
    assert rel(la.trsm(Fj, buf, lower=lower, out=buf, workspace=none), ref) <= TOL[dtype]
    Y, Lbar = la.trsm_backward(Fj, torch.from_numpy(ref.astype(NP[dtype])).cuda(), torch.from_numpy(Xbar).cuda(), lower=lower, workspace=none)
    Yref = np.linalg.solve(M.transpose(0, 2, 1), Xbar.astype(np.float64))
    assert rel(Y, Yref) <= TOL[dtype]
    G = -Yref @ ref.transpose(0, 2, 1)
    assert rel(Lbar, np.tril(G) if lower else np.triu(G)) <= TOL[dtype]


@pytest.mark.parametrize("batch,n,m", [(11700, 47, 8), (10700, 46, 45), (10700, 46, 40)])
def test_sizes_from_memory(batch, n, m):
    """potri of nearly whole tiles and products with rows of an odd number of vectors, beyond 128 (192) MiB in fp64"""
    g = torch.Generator(device="cuda").manual_seed(n)
    L = torch.randn(batch, n, n, generator=g, device="cuda", dtype=torch.float64).tril_().mul_(0.5 / n**0.5)
    L.diagonal(dim1=1, dim2=2).copy_(1 + torch.rand(batch, n, generator=g, device="cuda", dtype=torch.float64))
    X = torch.randn(batch, n, m, generator=g, device="cuda", dtype=torch.float64)
    ref = torch.bmm(L, X)
    assert float((la.trmm(L, X) - ref).norm() / ref.norm()) <= TOL["f64"]
    buf = X.clone()
    assert float((la.trmm(L, buf, out=buf) - ref).norm() / ref.norm()) <= TOL["f64"]
    B = la.potri(L)
    assert torch.equal(B, B.mT)
    one = torch.bmm(L.mT.contiguous(), torch.bmm(B, L))
    assert float((one - torch.eye(n, device="cuda", dtype=torch.float64)).norm() / (batch * n) ** 0.5) <= TOL["f64"]
