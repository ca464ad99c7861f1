"""Products with one to eight columns: each operand layout on both sides of the lines where few blocks and long sums are split finer, rows that
do not fill a block, sums that do not fill a step.

Bound: a sum of k products in another order differs from the 64-bit one by at most about k eps |A| |B|; of normal entries that is below
2 sqrt(k) eps of the result's norm (a random walk), held here with a factor of four to spare."""
import numpy as np
import pytest
import torch

import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float32, torch.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n", [1, 3, 8])
@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("b,m,k", [
    (1, 9, 2047), (1, 9, 2048), (1, 17, 4097), (3, 40, 2500), (1, 1400, 2100), (1, 1361, 2112),  # k contiguous: from 2048 and 12 a block on
    (1, 65, 63), (1, 65, 64), (1, 1000, 65), (5, 33, 127), (1, 8200, 64), (1, 8191, 66), (1, 130, 700),  # transposed: from 64 and half a block on
])
def test_gemm2_thin(dt, n, ta, b, m, k):
    rng = np.random.default_rng(b + 7 * m + 11 * n + 13 * k)
    A = torch.from_numpy(rng.standard_normal((b, k, m) if ta else (b, m, k))).to("cuda", dt)
    for tb in (False, True):
        B = torch.from_numpy(rng.standard_normal((b, n, k) if tb else (b, k, n))).to("cuda", dt)
        C = la.gemm2(A, B, ta=ta, tb=tb, alpha=0.5).double().cpu()
        a, bb = A.double().cpu(), B.double().cpu()
        ref = 0.5 * ((a.mT if ta else a) @ (bb.mT if tb else bb))
        err = (C - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
        assert float(err.max()) <= 8 * k ** 0.5 * torch.finfo(dt).eps


@pytest.mark.parametrize("U,n,noise", [(128, 300, 0.1), (129, 200, 1e-2), (333, 900, 1e-3), (700, 1000, 0.1)])
def test_sgp_vector_solves(U, n, noise):
    """The criterion's vector solves in single precision against the same in double: phi and the gradient of the noise hold them directly.  Bound:
    rounding of the inputs and of the factorisations, eps times the condition number of Kuu (its diagonal's shift bounds it by U / 0.1 + 1), eight
    times."""
    g = torch.Generator(device="cuda").manual_seed(U)
    Z, X = (4 * torch.rand(q, 4, generator=g, device="cuda", dtype=torch.float64) - 2 for q in (U, n))

    def rbf(P, Q):
        return torch.exp(-0.5 * torch.cdist(P, Q) ** 2)

    Kuu = rbf(Z, Z)
    Kuu.diagonal().add_(0.1)
    Kuu, Kuf = (0.5 * (Kuu + Kuu.mT)).float(), rbf(Z, X).float()
    diag, y = torch.ones(n, device="cuda"), torch.randn(n, generator=g, device="cuda", dtype=torch.float64).float()
    got = la.sgp_criterion(Kuu.contiguous(), Kuf.contiguous(), diag, y, noise)
    ref = la.sgp_criterion(Kuu.double().contiguous(), Kuf.double().contiguous(), diag.double(), y.double(), noise)
    for name in ("phi", "noise_bar", "y_bar"):
        err = (got[name].double() - ref[name]).norm() / ref[name].norm()
        assert float(err) <= 8 * torch.finfo(torch.float32).eps * (U / 0.1 + 1), name
