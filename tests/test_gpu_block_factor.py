"""The one-workgroup factorisation of a block of up to 128 rows at the edges of its 16 x 16 tiles: every number of
tile rows, whole and ragged, both triangles, in place, with a failing pivot in every part of a tile."""
import numpy as np
import pytest
import torch

import oracle
import paper_1710_08717_amd as la

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-10, "f32": 2e-4}
NP = {"f64": np.float64, "f32": np.float32}
SIZES = [65, 79, 80, 81, 95, 96, 97, 112, 113, 127, 128]


def spd(batch, n, seed, dtype):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((batch, n, 2 * n))
    return (X @ X.transpose(0, 2, 1) / (2 * n) + np.eye(n)).astype(NP[dtype])


def rel(x, ref):
    x = x.cpu().numpy().astype(np.float64).reshape(x.shape[0], -1)
    ref = ref.reshape(ref.shape[0], -1)
    return np.max(np.linalg.norm(x - ref, axis=1) / np.linalg.norm(ref, axis=1))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("n", SIZES)
def test_factor_in_place_with_junk_in_the_other_triangle(n, lower, dtype):
    A = spd(2, n, n, dtype)
    ref = oracle.potrf(A.astype(np.float64))
    junk = A.copy()
    junk[:, ~np.tril(np.ones((n, n), bool)) if lower else np.triu(np.ones((n, n), bool)) == 0] = np.nan
    buf = torch.from_numpy(junk).cuda()
    L = la.potrf(buf, lower=lower, out=buf)
    assert rel(L, ref if lower else ref.transpose(0, 2, 1)) <= TOL[dtype]
    other = L.triu(1) if lower else L.tril(-1)
    assert torch.count_nonzero(other) == 0


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [256 + 1, 256 + 16, 384, 384 - 15])
def test_blocks_with_their_inverses(n, dtype):
    """several blocks: the rows below are products with the inverse of each block's factor"""
    A = spd(3, n, n, dtype)
    assert rel(la.potrf(torch.from_numpy(A).cuda()), oracle.potrf(A.astype(np.float64))) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [66, 128])
def test_first_failing_pivot(n, dtype):
    bad = sorted({0, 1, 3, 4, 15, 16, 17, 31, 47, 48, 63, 64, 65, n - 1})
    A = spd(len(bad) + 1, n, 3, dtype)
    for b, k in enumerate(bad):
        A[b, k, k] = -1.0
    info = torch.zeros(len(A), dtype=torch.int32, device="cuda")
    L = la.potrf(torch.from_numpy(A).cuda(), info=info)
    assert info.cpu().tolist() == [k + 1 for k in bad] + [0]
    assert rel(L[-1:], oracle.potrf(A[-1:].astype(np.float64))) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lower", [True, False])
@pytest.mark.parametrize("pivot", [0.0, -1.0, float("nan")])
@pytest.mark.parametrize("batch,n", [(20, 66), (20, 100), (20, 128), (20, 300), (1539, 37), (1539, 64), (1100, 48), (1100, 64)])
def test_columns_before_a_failing_pivot(batch, n, pivot, lower, dtype):
    """the factor is unspecified from the failing column on, and right before it: in the failing tile, below it and in later blocks"""
    bad = sorted({1, 2, 3, 5, 8, 12, 15, 17, 24, 31, 33, 36, 40, 47, 63, 65, 80, 99, 127, 128, 131, 200, 257, n - 1})
    bad = [k for k in bad if k < n]
    A = np.repeat(spd(1, n, 11, "f64"), max(batch, len(bad)), axis=0)
    for b, k in enumerate(bad):
        A[b, k, :] = A[b, :, k] = 0.0
        A[b, k, k] = pivot
    info = torch.zeros(len(A), dtype=torch.int32, device="cuda")
    L = la.potrf(torch.from_numpy(A.astype(NP[dtype])).cuda(), lower=lower, info=info).cpu().numpy().astype(np.float64)
    L = L if lower else L.transpose(0, 2, 1)
    assert info[: len(bad)].tolist() == [k + 1 for k in bad] and not info[len(bad) :].any()
    for b, k in enumerate(bad):
        lead = np.linalg.cholesky(A[b, :k, :k])
        ref = np.vstack([lead, np.linalg.solve(lead, A[b, k:, :k].T).T])
        assert np.linalg.norm(L[b, :, :k] - ref) <= TOL[dtype] * np.linalg.norm(ref), k


@pytest.mark.parametrize("exponent", [-480, 480])
def test_scales_far_from_one(exponent):
    """the factor of 4^e A is 2^e times that of A, down to pivots of 2^-960"""
    A = torch.from_numpy(spd(1, 100, 7, "f64")).cuda()
    L = la.potrf(A)
    scaled = torch.ldexp(la.potrf(torch.ldexp(A, torch.tensor(2 * exponent, device="cuda"))), torch.tensor(-exponent, device="cuda"))
    assert (L - scaled).norm() <= 1e-13 * L.norm()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 15, 17, 33, 64, 65, 113, 128])
def test_criterion_of_every_number_of_tile_rows(n, dtype):
    A = spd(3, n, 50 + n, dtype)
    y = np.random.default_rng(n).standard_normal((3, n)).astype(NP[dtype])
    loss, grad = la.gp_criterion(torch.from_numpy(A).cuda(), torch.from_numpy(y).cuda())
    A, y = A.astype(np.float64), y.astype(np.float64)
    Ai = np.linalg.inv(A)
    a = np.einsum("bij,bj->bi", Ai, y)
    ref = 0.5 * (y * a).sum(1) + 0.5 * np.linalg.slogdet(A)[1]
    assert np.all(np.abs(loss.cpu().numpy() - ref) <= TOL[dtype] * (1 + np.abs(ref)))
    assert rel(grad, 0.5 * (Ai - a[:, :, None] * a[:, None, :])) <= TOL[dtype]
    assert torch.equal(grad, grad.transpose(1, 2))
