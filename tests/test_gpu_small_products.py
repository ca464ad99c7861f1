"""Products of many small matrices in one workgroup each, and the inverse's backward rule on them: the edges of the
16 x 16 tiles, operands off the 16-byte grid, NaN around the operands, and the sizes next to the rule's limits."""
import pytest
import torch

import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu

EPS = {torch.float32: 2.0 ** -23, torch.float64: 2.0 ** -52}


def _operand(g, dt, b, r, c, off):
    """b x r x c on the GPU, starting `off` elements behind a 16-byte boundary, NaN before and behind it."""
    buf = torch.full((b * r * c + 16,), float("nan"), dtype=dt, device="cuda")
    v = buf[4 + off:4 + off + b * r * c].view(b, r, c)
    v.copy_(torch.randn(b, r, c, generator=g, dtype=torch.float64))
    return v


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("m,n,k", [
    (4, 4, 33), (3, 40, 20), (5, 64, 1), (16, 16, 17), (17, 33, 16), (37, 32, 37), (33, 31, 48), (48, 48, 48),
    (64, 48, 33), (63, 49, 15), (20, 20, 80), (4, 7, 128), (15, 17, 129),
])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
def test_gemm2_small(dt, m, n, k, ta, tb):
    g = torch.Generator().manual_seed(m + 101 * n + 10007 * k)
    for b, off in ((255, 0), (256, 1), (259, 3)):
        A = _operand(g, dt, b, *((k, m) if ta else (m, k)), off)
        B = _operand(g, dt, b, *((n, k) if tb else (k, n)), off)
        C = la.gemm2(A, B, ta=bool(ta), tb=bool(tb), alpha=-1.5)
        a, bb = A.double().cpu(), B.double().cpu()
        a, bb = (a.mT.contiguous() if ta else a), (bb.mT.contiguous() if tb else bb)
        # k products and sums of one rounding each, and the factor
        bound = 1.5 * (k + 2) * EPS[dt] * torch.matmul(a.abs(), bb.abs())
        assert ((C.double().cpu() + 1.5 * torch.matmul(a, bb)).abs() <= bound).all(), (b, off)


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n", [17, 32, 33, 48, 49])
@pytest.mark.parametrize("lower", [True, False])
def test_potri_backward_small(dt, n, lower):
    """B and Bbar without any symmetry; only the factor's triangle is read."""
    g = torch.Generator().manual_seed(n)
    for b in (63, 64, 1030):
        B, G = _operand(g, dt, b, n, n, 1), _operand(g, dt, b, n, n, 2)
        T = torch.randn(b, n, n, generator=g, dtype=torch.float64).tril(-1) / n + 2 * torch.eye(n, dtype=torch.float64)
        L = T.to(dt).cuda()
        keep = torch.ones(n, n, dtype=torch.bool, device="cuda")
        keep = keep.tril() if lower else keep.triu()
        Lin = torch.where(keep, L if lower else L.mT, torch.full_like(L, float("nan"))).contiguous()
        out = la.potri_backward(Lin, B, G, lower=lower).double().cpu()
        l, bb, S = L.double().cpu(), B.double().cpu(), G.double().cpu()
        S = S + S.mT
        Sa = G.double().cpu().abs()
        Sa = Sa + Sa.mT
        li = torch.linalg.inv(l)
        lit = li.mT.contiguous()
        amp = torch.matmul(torch.matmul(lit.abs(), l.mT.abs().contiguous()), lit.abs())
        if lower:  # -tril(B S L^-T)
            ref, bound = -torch.matmul(torch.matmul(bb, S), lit).tril(), torch.matmul(torch.matmul(bb.abs(), Sa), amp)
        else:      # -triu(R^-T S B) = -triu(L^-1 S B)
            ref = -torch.matmul(li, torch.matmul(S, bb)).triu()
            bound = torch.matmul(amp.mT.contiguous(), torch.matmul(Sa, bb.abs()))
        # n sums each in the product and in the substitution, one rounding of G + G^T
        assert ((out - ref).abs() <= (3 * n + 4) * EPS[dt] * bound).all(), b
