"""Products of many small matrices in one workgroup each: the edges of the
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
