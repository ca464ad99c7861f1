"""The factorisation's gradient swept block column by block column, at the edges of the block rule: last blocks of one row and of
nearly a whole block, every block size, both triangles, in place, beside the problems just below the rule; and operators whose inner
dimension is a multiple of 16 but not of 64."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08717_amd as la
from paper_1710_08717_amd import binding

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 2e-4}
NP = {"f64": np.float64, "f32": np.float32}


def rel(x, ref):
    x = x.cpu().numpy().astype(np.float64).reshape(x.shape[0], -1)
    ref = np.asarray(ref).reshape(ref.shape[0], -1)
    return np.max(np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1))


def factor(batch, n, rng, dtype):
    L = np.tril(rng.standard_normal((batch, n, n))) * (0.5 / np.sqrt(n))
    i = np.arange(n)
    L[:, i, i] = 1.0 + rng.random((batch, n))
    return L.astype(NP[dtype])


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n", [(400, 257), (300, 214), (600, 214), (280, 213), (129, 400), (53, 400), (36, 513), (8, 770), (13, 799), (9, 1025), (4, 1024), (3, 1183), (2, 2048)])
def test_sweep(batch, n, lower, dtype):
    rng = np.random.default_rng(n)
    L = factor(batch, n, rng, dtype)
    Lbar = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    if not lower:
        L = L.transpose(0, 2, 1).copy()
    ref = oracle.potrf_backward(L.astype(np.float64), Lbar.astype(np.float64), lower=lower)
    other = np.triu(np.ones((n, n), bool), 1) if lower else np.tril(np.ones((n, n), bool), -1)
    L[:, other] = np.nan
    Lbar[:, other] = np.nan
    Lg, Gg = torch.from_numpy(L).cuda(), torch.from_numpy(Lbar).cuda()
    got = la.potrf_backward(Lg, Gg, lower=lower)
    assert torch.equal(got, got.mT)
    assert rel(got, ref) <= TOL[dtype]
    inplace = la.potrf_backward(Lg, Gg, lower=lower, out=Gg)
    assert torch.equal(inplace, got)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("batch,n", [(1, 144), (3, 208), (2, 336), (1, 720), (40, 304)])
def test_inner_dimension_of_16_not_64(batch, n, dtype):
    rng = np.random.default_rng(n)
    L = factor(batch, n, rng, dtype)
    X = rng.standard_normal((batch, n, 48)).astype(NP[dtype])
    G = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    L64, X64, G64 = (np.tril(L).astype(np.float64), X.astype(np.float64), G.astype(np.float64))
    Lg, Xg, Gg = (torch.from_numpy(x).cuda() for x in (L, X, G))
    assert rel(la.trmm(Lg, Xg), L64 @ X64) <= TOL[dtype]
    assert rel(la.gemm2(Gg, Xg), G64 @ X64) <= TOL[dtype]
    assert rel(la.syrk_backward(Xg, Gg), (G64 + G64.transpose(0, 2, 1)) @ X64) <= TOL[dtype]
    assert rel(la.potri(Lg), oracle.potri(L64)) <= TOL[dtype]
    assert rel(la.potrf_backward(Lg, Gg), oracle.potrf_backward(L64, G64)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n,k", [(64, 128, 128), (63, 129, 131), (64, 127, 128), (5, 517, 127), (5, 517, 160)])
def test_rules_on_the_symmetric_sum(batch, n, k, lower, dtype):
    """potri's and syrk's backward rules on both sides of the sizes from which G + G^T is formed"""
    rng = np.random.default_rng(n + k)
    L = factor(batch, n, rng, dtype)
    G = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    A = rng.standard_normal((batch, n, k) if lower else (batch, k, n)).astype(NP[dtype])
    if not lower:
        L = L.transpose(0, 2, 1).copy()
    B = oracle.potri(L.astype(np.float64), lower=lower).astype(NP[dtype])
    Lg, Gg, Ag, Bg = (torch.from_numpy(x).cuda() for x in (L, G, A, B))
    ref = oracle.potri_backward(L.astype(np.float64), B.astype(np.float64), G.astype(np.float64), lower=lower)
    assert rel(la.potri_backward(Lg, Bg, Gg, lower=lower), ref) <= TOL[dtype]
    S = G.astype(np.float64) + G.transpose(0, 2, 1).astype(np.float64)
    ref = S @ A.astype(np.float64) if lower else A.astype(np.float64) @ S
    assert rel(la.syrk_backward(Ag, Gg, trans=not lower), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("batch,n", [(3, 214), (2, 300), (3, 513), (70, 500), (5, 1025), (2, 1183), (1, 2300)])
def test_sweep_on_short_workspaces(batch, n, lower, dtype):
    """fewer inverses at a time and smaller blocks: from the full workspace down to the least, in place and not, nothing behind it touched"""
    rng = np.random.default_rng(n)
    L = factor(batch, n, rng, dtype)
    Lbar = rng.standard_normal((batch, n, n)).astype(NP[dtype])
    if not lower:
        L = L.transpose(0, 2, 1).copy()
    ref = oracle.potrf_backward(L.astype(np.float64), Lbar.astype(np.float64), lower=lower)
    other = np.triu(np.ones((n, n), bool), 1) if lower else np.tril(np.ones((n, n), bool), -1)
    L[:, other] = np.nan
    Lbar[:, other] = np.nan
    Lg, Gg = torch.from_numpy(L).cuda(), torch.from_numpy(Lbar).cuda()
    full = la.workspace_bytes(binding.OP_POTRF_BACKWARD, Lg, batch, n)
    least = batch * (3 * 128 * 128 + 128) * Lg.element_size()
    assert least < full
    for need in sorted({least, full} | {least + (full - least) * q // 8 // 256 * 256 for q in range(8)}):
        buf = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        got = la.potrf_backward(Lg, Gg, lower=lower, workspace=buf[:need])
        assert torch.equal(got, got.mT), need
        assert rel(got, ref) <= TOL[dtype], need
        inplace = Gg.clone()
        assert torch.equal(la.potrf_backward(Lg, inplace, lower=lower, out=inplace, workspace=buf[:need]), got), need
        assert (buf[need:] == 0xA5).all(), need
    with pytest.raises(la.LaError):
        la.potrf_backward(Lg, Gg, lower=lower, workspace=buf[:least - 256])


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("batch,m,n,k", [(25, 256, 256, 144), (28, 256, 256, 208), (103, 128, 128, 400), (112, 128, 128, 400), (513, 64, 64, 272),
                                         (150, 64, 256, 336), (137, 80, 160, 176), (255, 128, 128, 144), (64, 96, 300, 1040)])
def test_products_on_both_sides_of_the_tile_rule(batch, m, n, k, dtype):
    """aligned operands, inner dimension a multiple of 16 but not of 64: tiles of 64 and quarter tiles, uniform, triangular and symmetric"""
    g = torch.Generator(device="cuda").manual_seed(batch)
    dt = torch.float64 if dtype == "f64" else torch.float32
    R = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=dt)
    err = lambda x, r: float((x.double() - r).norm() / r.norm())
    A, B = R(batch, m, k), R(batch, k, n)
    At, Bt = A.mT.contiguous(), B.mT.contiguous()
    ref = torch.bmm(A.double(), B.double())
    for ta in (False, True):
        for tb in (False, True):
            assert err(la.gemm2(At if ta else A, Bt if tb else B, ta=ta, tb=tb), ref) <= TOL[dtype]
    assert err(la.syrk(A), torch.bmm(A.double(), At.double())) <= TOL[dtype]
    L = R(batch, k, k).tril_()
    assert err(la.trmm(L, B), torch.bmm(L.double(), B.double())) <= TOL[dtype]
    assert err(la.trmm(L, A, rightside=True), torch.bmm(A.double(), L.double())) <= TOL[dtype]
