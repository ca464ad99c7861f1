"""Products whose sizes and leading dimensions are no multiple of a vector or of a tile: the chunks that cross the
end of an operand, in each operand layout, at the edges of the 16 / 32 / 64 tiles and of the K slabs, and in 128 x 128 tiles."""
import numpy as np
import pytest
import torch

import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu

TOL = {torch.float32: 2e-4, torch.float64: 1e-10}


def _operand(rng, dt, b, r, c, off):
    """b x r x c on the GPU, starting `off` elements behind a 16-byte boundary, NaN before and behind it."""
    buf = torch.full((b * r * c + 16,), float("nan"), dtype=dt, device="cuda")
    v = buf[4 + off:4 + off + b * r * c].view(b, r, c)
    v.copy_(torch.from_numpy(rng.standard_normal((b, r, c))))
    return v


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,m,n,k", [
    (1, 33, 34, 1), (3, 37, 41, 15), (2, 63, 65, 17), (9, 65, 33, 31), (2, 127, 129, 33), (1, 129, 127, 63),
    (1, 131, 257, 65), (17, 61, 67, 127), (1, 333, 97, 129), (2, 1025, 1023, 50), (1, 1667, 1793, 77),
    (1, 35, 45, 4099),
])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm2_ragged(dt, b, m, n, k, ta, tb):
    rng = np.random.default_rng(b + 7 * m + 11 * n + 13 * k)
    for off in (0, 1):
        A = _operand(rng, dt, b, *((k, m) if ta else (m, k)), off)
        B = _operand(rng, dt, b, *((n, k) if tb else (k, n)), off)
        C = la.gemm2(A, B, ta=bool(ta), tb=bool(tb))
        a, bb = A.double().cpu(), B.double().cpu()
        ref = torch.matmul(a.mT.contiguous() if ta else a, bb.mT.contiguous() if tb else bb)
        err = (C.double().cpu() - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
        assert float(err.max()) <= TOL[dt], (off, float(err.max()))


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("cols", range(1, 10))
@pytest.mark.parametrize("m,k", [(200, 5), (70, 131), (9, 1025)])
def test_thin_products(dt, cols, m, k):
    """One instance of the kernel per number of columns up to eight, plain and with a triangular operand."""
    for ta, tb in ((0, 0), (0, 1), (1, 0), (1, 1)):
        test_gemm2_ragged(dt, 3, m, cols, k, ta, tb)
        test_gemm2_ragged(dt, 3, cols, m, k, ta, tb)
    for trans in (0, 1):
        test_trmm_big_tiles(dt, 2, 140 + m, cols, 1, trans)


# (b, m, n, k): with K above 32, 128 x 128 tiles are taken from 480 of them on, if they stick out of C by less than a quarter more than tiles of
# 64 do; in fp64, aligned and with k not contiguous in both operands, also for 225 to 256 of them (193 in a batch).
BIG_TILES = [(130, 255, 253, 33), (130, 254, 255, 35), (55, 383, 381, 77), (33, 509, 511, 130), (13, 512, 512, 64),
             (64, 256, 256, 48), (1, 1920, 1920, 48)]


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,m,n,k", BIG_TILES)
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm2_big_tiles(dt, b, m, n, k, ta, tb):
    t128, t64 = -(-m // 128) * -(-n // 128), -(-m // 64) * -(-n // 64)
    one_round = m % 2 == 0 and n % 2 == 0 and k % 16 == 0 and (192 if b > 1 else 224) < b * t128 <= 256
    assert k > 32 and 16 * t128 <= 5 * t64 and (b * t128 >= 480 or one_round)
    test_gemm2_ragged(dt, b, m, n, k, ta, tb)


# next to the rules that keep 64 x 64 tiles: K up to 32 where there are enough big ones, and ragged products of 960 tiles and more
@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,m,n,k", [(130, 254, 255, 15), (64, 256, 256, 16), (1, 1920, 1920, 32),
                                     (130, 254, 255, 32), (55, 383, 381, 1), (319, 61, 174, 147),
                                     (320, 61, 174, 147), (331, 63, 187, 255), (26, 2478, 22, 130)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm2_kept_tiles(dt, b, m, n, k, ta, tb):
    test_gemm2_ragged(dt, b, m, n, k, ta, tb)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,n,m", [(257, 255, 253), (260, 254, 251), (600, 129, 130)])
@pytest.mark.parametrize("lower,trans", [(1, 0), (0, 0), (1, 1)])
def test_trmm_big_tiles(dt, b, n, m, lower, trans):
    """A masked operand in 128 x 128 tiles (from 1024 of them on) and, at n = 129, in the smaller ones that replace them."""
    rng = np.random.default_rng(n + m)
    L, X = _operand(rng, dt, b, n, n, 1), _operand(rng, dt, b, n, m, 0)
    Y = la.trmm(L, X, lower=bool(lower), trans=bool(trans))
    t = L.double().tril() if lower else L.double().triu()
    ref = torch.matmul((t.mT if trans else t).contiguous(), X.double())
    err = (Y.double() - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
    assert float(err.max()) <= TOL[dt], float(err.max())


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("b,n", [(1, 129), (3, 191), (2, 257), (1, 515), (1, 1031), (1, 2307)])
def test_triangular_ragged(dt, b, n):
    """Masked operands, masked and mirrored results: factor, gradient of the factor, inverse."""
    g = torch.Generator().manual_seed(n)
    X = torch.randn(b, n, n + 8, generator=g, dtype=torch.float64)
    A = torch.matmul(X, X.mT.contiguous()) / n + torch.eye(n, dtype=torch.float64)
    G = torch.randn(b, n, n, generator=g, dtype=torch.float64)
    Ad, Gd = A.to(dt).cuda(), G.to(dt).cuda()
    for lower in (True, False):
        L = la.potrf(Ad, lower=lower)
        Abar = la.potrf_backward(L, Gd, lower=lower)
        Ainv = la.potri(L, lower=lower)
        A64, G64 = Ad.double().cpu(), Gd.double().cpu()
        Lr = torch.linalg.cholesky(A64)
        Gr = (G64 if lower else G64.mT).tril()
        P = torch.matmul(Lr.mT.contiguous(), Gr).tril()
        P = P + P.tril(-1).mT
        W = torch.linalg.solve_triangular(Lr.mT, P, upper=True)
        W = torch.linalg.solve_triangular(Lr, W, upper=False, left=False)
        ref = {"L": Lr if lower else Lr.mT, "Abar": 0.25 * (W + W.mT), "Ainv": torch.cholesky_inverse(Lr)}
        for name, got in (("L", L), ("Abar", Abar), ("Ainv", Ainv)):
            err = (got.double().cpu() - ref[name]).flatten(1).norm(dim=1) / ref[name].flatten(1).norm(dim=1)
            assert float(err.max()) <= TOL[dt], (name, lower, float(err.max()))
