"""Parity of la_kalman_filter (section 3.4) against the oracle's filter on the same seeded
synthetic sequences.  The recursion is contractive here (stable transition matrix, every step
conditions on a new observation), so rounding errors do not build up over the steps and the
operators' tolerance applies to every output; the likelihood is a sum of T terms of size O(dv)
and is compared relative to its value."""
import sys

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = {"f32": 2e-4, "f64": 1e-10}


@pytest.fixture(scope="module")
def la():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1710_08717_amd as la_mod

    la_mod.load()
    return la_mod


@pytest.fixture(autouse=True)
def _announce(request):
    sys.stderr.write(f"\n[gpu-case] {request.node.nodeid}\n")
    sys.stderr.flush()
    yield


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, dtype=np.float64) - b) / max(np.linalg.norm(b), 1e-300))


def run(la, w, want_states=True, with_info=True):
    import torch

    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    info = torch.full((w["batch"],), -1, dtype=torch.int32, device="cuda") if with_info else None
    nll, f, F = la.kalman_filter(dev(w["A"]), dev(w["B"]), dev(w["Sh"]), dev(w["Sv"]), dev(w["mu0"]), dev(w["S0"]),
                                 dev(w["v"]), want_states=want_states, info=info)
    torch.cuda.synchronize()
    host = lambda t: None if t is None else t.cpu().numpy()
    return host(nll), host(f), host(F), host(info)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("shared", [True, False])
@pytest.mark.parametrize("batch,T,dh,dv", [(1, 1, 1, 1), (3, 5, 2, 1), (5, 7, 3, 5), (9, 12, 4, 4), (6, 9, 7, 3),
                                           (4, 20, 16, 16), (7, 6, 16, 5), (5, 6, 5, 16), (130, 8, 8, 8),
                                           (5, 7, 5, 8), (11, 6, 8, 5), (2, 0, 3, 2)])
def test_kalman_parity(la, orc, dtype, shared, batch, T, dh, dv):
    w = workloads.make_kalman(batch, T, dh, dv, dtype=dtype, shared=shared, seed=batch + T)
    ref_nll, ref_f, ref_F, ref_info = orc.kalman_filter(w["A"], w["B"], w["Sh"], w["Sv"], w["mu0"], w["S0"], w["v"])
    nll, f, F, info = run(la, w)
    tol = TOL[dtype]
    assert np.array_equal(info, ref_info) and np.all(info == 0)
    assert np.all(np.abs(nll - ref_nll) <= tol * np.maximum(1.0, np.abs(ref_nll)))
    if T > 0:
        assert rel(f, ref_f) <= tol
        assert rel(F, ref_F) <= tol
        # per sequence and step as well, so that one bad item cannot hide in the norm of many
        per = np.linalg.norm((F - ref_F).reshape(batch, T, -1), axis=2) / np.linalg.norm(ref_F.reshape(batch, T, -1), axis=2)
        assert per.max() <= tol
    # likelihood only: same value, no state outputs written
    nll2, f2, F2, _ = run(la, w, want_states=False, with_info=False)
    assert f2 is None and F2 is None
    assert np.array_equal(nll2, nll)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_kalman_many_long_sequences(la, orc, dtype):
    """Thousands of workgroups and a few hundred steps; a batch that is no multiple of the four
    sequences a workgroup carries."""
    w = workloads.make_kalman(4099, 64, 6, 4, dtype=dtype, shared=True, seed=11)
    ref_nll, ref_f, ref_F, _ = orc.kalman_filter(w["A"], w["B"], w["Sh"], w["Sv"], w["mu0"], w["S0"], w["v"])
    nll, f, F, info = run(la, w)
    tol = TOL[dtype]
    assert np.all(info == 0)
    assert np.all(np.abs(nll - ref_nll) <= tol * np.maximum(1.0, np.abs(ref_nll)))
    assert rel(f, ref_f) <= tol and rel(F, ref_F) <= tol
    w = workloads.make_kalman(3, 400, 16, 8, dtype=dtype, shared=False, seed=12)
    ref_nll, ref_f, ref_F, _ = orc.kalman_filter(w["A"], w["B"], w["Sh"], w["Sv"], w["mu0"], w["S0"], w["v"])
    nll, f, F, info = run(la, w)
    assert np.all(np.abs(nll - ref_nll) <= tol * np.maximum(1.0, np.abs(ref_nll)))
    assert rel(f[:, -1], ref_f[:, -1]) <= tol and rel(F[:, -1], ref_F[:, -1]) <= tol


@pytest.mark.parametrize("dtype,dh,dv", [("f64", 3, 2), ("f32", 7, 6), ("f32", 12, 9)])  # 4, 8 and 16 lanes per sequence
def test_kalman_reports_a_failing_pivot(la, orc, dtype, dh, dv):
    w = workloads.make_kalman(6, 5, dh, dv, dtype=dtype, shared=False, seed=3)
    w["Sv"][4] = -50.0 * np.eye(dv)  # sequence 4: S_vv is not positive definite from the first step on
    _, _, _, ref_info = orc.kalman_filter(w["A"], w["B"], w["Sh"], w["Sv"], w["mu0"], w["S0"], w["v"])
    nll, f, F, info = run(la, w)
    assert np.array_equal(info, ref_info) and info[4] == 1 and np.all(np.delete(info, 4) == 0)
    ok = np.delete(np.arange(6), 4)
    ref = orc.kalman_filter(w["A"][ok], w["B"][ok], w["Sh"][ok], w["Sv"][ok], w["mu0"][ok], w["S0"][ok], w["v"][ok])
    assert np.all(np.abs(nll[ok] - ref[0]) <= TOL[dtype] * np.maximum(1.0, np.abs(ref[0])))


def test_kalman_argument_errors(la):
    import ctypes

    import torch

    lib = la.load()
    x = torch.zeros(64, dtype=torch.float32, device="cuda")
    p = ctypes.c_void_p(x.data_ptr())
    z = ctypes.c_void_p(0)
    args = lambda dh, dv, nll: (0, 1, 1, dh, dv, 1, p, p, p, p, p, p, p, z, z, nll, z, z)
    assert lib.la_kalman_filter(*args(17, 2, p)) == 2   # LA_ERR_UNSUPPORTED
    assert lib.la_kalman_filter(*args(2, 17, p)) == 2
    assert lib.la_kalman_filter(*args(0, 2, p)) == 1    # LA_ERR_INVALID_ARG
    assert lib.la_kalman_filter(*args(2, 2, z)) == 1
    assert lib.la_kalman_filter(7, 1, 1, 2, 2, 1, p, p, p, p, p, p, p, z, z, p, z, z) == 1
    assert lib.la_kalman_filter(0, 0, 1, 2, 2, 1, z, z, z, z, z, z, z, z, z, z, z, z) == 0  # empty batch


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("batch,T,dh,dv", [(31, 4, 16, 16), (33, 3, 15, 9), (65, 3, 11, 12), (17, 5, 12, 1), (40, 2, 4, 13),
                                           (32768 + 37, 2, 9, 3), (32768 + 33, 3, 3, 8), (1, 9, 1, 16)])
@pytest.mark.parametrize("want_states", [True, False])
def test_kalman_one_model_equals_repeated_model(la, dtype, batch, T, dh, dv, want_states):
    """The kernel that shares the covariance recursion against the per-sequence one on the same model, repeated:
    covariances that are not symmetric (read as they are), ends of the 16-sequence tiles, F items of odd size."""
    w = workloads.make_kalman(batch, T, dh, dv, dtype=dtype, shared=True, seed=batch + 3 * T)
    g = np.random.default_rng(batch)
    for k in ("Sh", "S0"):
        w[k] = (w[k] + 0.01 * g.standard_normal(w[k].shape)).astype(w[k].dtype)
    rep = dict(w)
    for k in ("A", "B", "Sh", "Sv", "mu0", "S0"):
        rep[k] = np.repeat(w[k][None], batch, axis=0)
    a, b = run(la, w, want_states), run(la, rep, want_states)
    assert np.array_equal(a[3], b[3])
    assert np.all(np.abs(a[0] - b[0]) <= TOL[dtype] * np.maximum(1.0, np.abs(b[0])))
    if want_states:
        assert rel(a[1], b[1]) <= TOL[dtype] and rel(a[2], b[2]) <= TOL[dtype]


def test_kalman_one_model_bad_pivot(la):
    """info and the step a pivot fails at, shared against repeated parameters."""
    w = workloads.make_kalman(20, 4, 5, 3, dtype="f64", shared=True, seed=3)
    w["Sv"] = -50.0 * np.eye(3)
    rep = dict(w)
    for k in ("A", "B", "Sh", "Sv", "mu0", "S0"):
        rep[k] = np.repeat(w[k][None], 20, axis=0)
    assert np.array_equal(run(la, w)[3], run(la, rep)[3])
    assert np.all(run(la, w)[3] == 1)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dh,dv", [(5, 3), (2, 4), (16, 16)])
def test_kalman_one_model_pivot_of_a_later_step(la, dtype, dh, dv):
    """An indefinite state noise makes one variance negative after some steps: info names the first step whose S_vv is not
    positive definite (its least eigenvalue is 0.1 the step before and -8 there), in both kernels, and no later one."""
    w = workloads.make_kalman(20, 9, dh, dv, dtype=dtype, shared=True, seed=3)
    w["A"], w["B"], w["Sv"] = np.eye(dh), np.eye(dv, dh), np.eye(dv)
    w["Sh"], w["S0"] = np.diag(np.where(np.arange(dh) == 1, -0.9, 0.1)), 10.0 * np.eye(dh)
    S, first = w["S0"], 0
    for t in range(9):
        if t > 0:
            S = F + w["Sh"]
        Svv = w["B"] @ S @ w["B"].T + w["Sv"]
        if np.linalg.eigvalsh(Svv)[0] <= 0:
            first = t + 1
            break
        F = S - S @ w["B"].T @ np.linalg.solve(Svv, w["B"] @ S)
    assert first == 4
    for k in ("A", "B", "Sh", "Sv", "S0"):
        w[k] = w[k].astype(workloads.np_dtype(dtype))
    rep = dict(w)
    for k in ("A", "B", "Sh", "Sv", "mu0", "S0"):
        rep[k] = np.repeat(w[k][None], 20, axis=0)
    assert np.all(run(la, w)[3] == first) and np.all(run(la, rep)[3] == first)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("batch,dh,dv", [(8193, 4, 3), (8197, 2, 9), (16385, 7, 5), (16385, 16, 16)])
def test_kalman_one_model_with_32_sequences_a_wavefront(la, dtype, batch, dh, dv):
    """The split for batches of more workgroups than the chip holds, ragged at its end."""
    test_kalman_one_model_equals_repeated_model(la, dtype, batch, 3, dh, dv, True)


@pytest.mark.parametrize("batch,dh,dv,want", [(50, 1, 3, True), (37, 3, 4, False), (16387, 3, 2, True), (16401, 4, 4, False),
                                              (49155, 2, 4, True), (65539, 3, 3, True), (65551, 4, 4, True), (65537, 2, 2, False),
                                              (65543, 4, 5, True)])
def test_kalman_one_model_of_small_dimensions(la, batch, dh, dv, want):
    """fp32: one recursion per sequence or a common one by size, and up to 64 sequences per wavefront in the common one."""
    test_kalman_one_model_equals_repeated_model(la, "f32", batch, 3, dh, dv, want)


def _filter_80_bit(w):
    """Filtered means and covariances of one model over its sequences in 80-bit floats."""
    ld = np.longdouble
    A, B, Sh, Sv, mu, S, v = (w[k].astype(ld) for k in ("A", "B", "Sh", "Sv", "mu0", "S0", "v"))
    f, fs, Fs, eye = np.repeat(mu[None], len(v), 0), [], [], np.eye(len(A), dtype=ld)
    for t in range(v.shape[1]):
        if t > 0:
            f, S = f @ A.T, A @ F @ A.T + Sh
        X, M = B @ S @ B.T + Sv, (S @ B.T).T  # K^T = X^-1 M by elimination
        for k in range(len(X)):
            m = X[k + 1:, k:k + 1] / X[k, k]
            X[k + 1:], M[k + 1:] = X[k + 1:] - m * X[k], M[k + 1:] - m * M[k]
        for k in reversed(range(len(X))):
            M[k] = (M[k] - X[k, k + 1:] @ M[k + 1:]) / X[k, k]
        K = M.T
        f = f + (v[:, t] - f @ B.T) @ K.T
        F = (eye - K @ B) @ S @ (eye - K @ B).T + K @ Sv @ K.T
        fs.append(f)
        Fs.append(F)
    return np.stack(fs, 1), np.stack(Fs)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dh,dv", [(1, 16), (2, 16), (4, 16), (8, 16), (4, 4), (13, 9), (3, 7), (12, 13)])
def test_kalman_one_model_is_as_accurate_as_repeated_model(la, dtype, dh, dv):
    """Little observation noise makes S_vv ill-conditioned.  The gain of the shared recursion then has to be as accurate as
    the row-wise substitution of the per-sequence kernel: the mean error over ten models within 1.6 of its (two sums of
    roundings of the same size, in another order); from an explicit inverse it is 2 to 16 times as large for dv > dh."""
    errs = np.zeros((2, 2))
    for seed in range(10):
        w = workloads.make_kalman(12, 15, dh, dv, dtype=dtype, shared=True, seed=seed)
        w["Sv"] = (w["Sv"] * 1e-4).astype(w["Sv"].dtype)
        rep = dict(w)
        for k in ("A", "B", "Sh", "Sv", "mu0", "S0"):
            rep[k] = np.repeat(w[k][None], 12, axis=0)
        rf, rF = _filter_80_bit(w)
        for i, x in enumerate((w, rep)):
            _, f, F, _ = run(la, x)
            d, D = f.astype(np.longdouble) - rf, F[0].astype(np.longdouble) - rF
            errs[i] += [float(np.sqrt((d * d).sum() / (rf * rf).sum())), float(np.sqrt((D * D).sum() / (rF * rF).sum()))]
    sys.stderr.write(f"f {errs[0, 0] / errs[1, 0]:.2f} F {errs[0, 1] / errs[1, 1]:.2f}\n")
    assert errs[0, 0] <= 1.6 * errs[1, 0] and errs[0, 1] <= 1.6 * errs[1, 1]
