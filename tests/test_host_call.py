"""The binding's two ways to the library: plain calls through csrc/host_call.cpp give what the ctypes calls give, bit for bit, and all other calls
are left to these."""
import os
import re
import shutil
import subprocess
import sys

import pytest
import torch

import paper_1710_08717_amd as la
from paper_1710_08717_amd import binding, build


def spd(batch, n, dt):
    X = torch.randn(batch, n, n, dtype=dt)
    return X @ X.mT + n * torch.eye(n, dtype=dt)


def calls(L, A, R, y):
    B = la.potri(L)
    return {
        "potrf": lambda: la.potrf(A), "potrf_u": lambda: la.potrf(A, lower=False), "potrf_b": lambda: la.potrf_backward(L, A),
        "trsm": lambda: la.trsm(L, R), "trsm_t": lambda: la.trsm(L, R, trans=True, alpha=0.5), "trsm_r": lambda: la.trsm(L, R.mT.contiguous(), rightside=True),
        "trmm": lambda: la.trmm(L, R), "trsm_b": lambda: la.trsm_backward(L, R, R), "trmm_b": lambda: la.trmm_backward(L, R, R, trans=True),
        "syrk": lambda: la.syrk(R), "syrk_t": lambda: la.syrk(R, trans=True, alpha=2.0), "syrk_b": lambda: la.syrk_backward(R, A),
        "gemm2": lambda: la.gemm2(R, A, ta=True), "gemm2_b": lambda: la.gemm2_backward(R, A, R.mT.contiguous(), ta=True),
        "potri": lambda: la.potri(L), "potri_b": lambda: la.potri_backward(L, B, A), "logdet": lambda: la.sumlogdiag(L),
        "gp": lambda: la.gp_criterion(A, y),
    }


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [torch.float32, torch.float64])
@pytest.mark.parametrize("lead,n,m", [((), 5, 3), ((0,), 4, 2), ((2, 3), 33, 7), ((2,), 300, 20)])
def test_both_ways_agree(dt, lead, n, m, monkeypatch):
    torch.manual_seed(n)
    b = 1
    for s in lead:
        b *= s
    A = spd(b, n, dt).reshape(*lead, n, n).cuda()
    R, y = torch.randn(*lead, n, m, dtype=dt).cuda(), torch.randn(*lead, n, dtype=dt).cuda()
    L = la.potrf(A)
    fast = {k: f() for k, f in calls(L, A, R, y).items()}
    monkeypatch.setattr(binding, "_host", None)
    for k, f in calls(L, A, R, y).items():
        for x, z in zip(*[(t if isinstance(t, tuple) else (t,)) for t in (fast[k], f())]):
            assert x.shape == z.shape and x.dtype == z.dtype and x.device == z.device and not x.requires_grad, k
            assert torch.equal(x, z), k


@pytest.mark.gpu
def test_other_calls_are_left_to_ctypes():
    host = la.load() and binding._host
    A = spd(2, 6, torch.float64).cuda()
    assert host.potrf(A, True) is not None
    for bad in ((A.mT, True), (A.half(), True), (A[:, :5], True), (A.cpu(), True), (A, 1), (A.tolist(), True), (A,),
                (A.to_sparse(), True)):
        assert host.potrf(*bad) is None
    assert host.tri(True, A, A.float(), True, False, False, 1.0) is None
    assert host.tri(True, A, A[:1], True, False, False, 1.0) is None
    assert host.tri(True, A, A, True, False, False, 1) is None
    assert host.gemm2(A, A[:, :5].contiguous(), False, False, 1.0) is None
    from torch.overrides import TorchFunctionMode

    with TorchFunctionMode():
        assert host.potrf(A, True) is None
    seen = []
    torch.func.vmap(lambda x: seen.append(host.potrf(x, True)) or x)(A)
    assert seen == [None]
    for fn in (lambda: la.potrf(A.mT), lambda: la.potrf(A.half()), lambda: la.trsm(A, A.float()), lambda: la.gemm2(A, A.cpu())):
        with pytest.raises(la.LaError):
            fn()
    with pytest.raises(AssertionError):
        la.trsm(A, A[:1].contiguous())
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        L = la.potrf(A)
    s.synchronize()
    assert torch.equal(L, la.potrf(A))


def test_host_call_leaves_cpu_tensors():
    la.load()
    A = torch.eye(3)[None]
    assert binding._host.potrf(A, True) is None and binding._host.gp_criterion(A, A[:, 0]) is None
    with pytest.raises(la.LaError):
        la.potrf(A)


TRANSFORMS = {
    "grad": lambda f, x: torch.func.grad(f)(x), "jvp": lambda f, x: torch.func.jvp(f, (x,), (x,)), "jacrev": lambda f, x: torch.func.jacrev(f)(x),
    "hessian": lambda f, x: torch.func.hessian(f)(x), "vmap": lambda f, x: torch.func.vmap(f)(x[:, None]),
    "functionalize": lambda f, x: torch.func.functionalize(f)(x),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", TRANSFORMS)
@pytest.mark.parametrize("n", [8, 300])  # without and with a workspace
def test_transforms_over_a_closed_over_tensor_go_by_ctypes(name, n):
    """grad and the like wrap what is allocated inside them: an error that names it, as ever, where the result has no storage; vmap does not"""
    torch.manual_seed(0)
    A, x = spd(2, n, torch.float64).cuda(), torch.ones(3, device="cuda", dtype=torch.float64)
    L, R, y = la.potrf(A), torch.randn(2, n, 3, dtype=torch.float64).cuda(), torch.randn(2, n, dtype=torch.float64).cuda()
    seen, raised = [], []

    def f(v):
        for k, c in table.items():
            try:
                seen.append((k, c()))
            except RuntimeError as e:
                raised.append((k, str(e)))
        return v.sum()

    table = calls(L, A, R, y)
    want = {k: c() for k, c in table.items()}
    TRANSFORMS[name](f, x)
    if name == "vmap":
        assert not raised
        for k, got in seen:
            for a, b in zip(*[(t if isinstance(t, tuple) else (t,)) for t in (got, want[k])]):
                assert torch.equal(a, b), k
    elif name != "functionalize":
        assert {k for k, _ in raised} == set(table) and all("storage" in e for _, e in raised), raised
    assert torch.equal(la.potrf(A), L)


# host_call.cpp with its device checks turned to the CPU, on a library whose functions do nothing: the paths that leave a call, without a GPU
CPU = [("t.is_cuda()", "t.is_cpu()"), ("DispatchKey::CUDA", "DispatchKey::CPU"), ("DispatchKey::AutogradCUDA", "DispatchKey::AutogradCPU"),
       ("DispatchKey::AutocastCUDA", "DispatchKey::AutocastCPU"), ("c10::hip::current_device()", "-1"),
       ("(void *)c10::hip::getCurrentHIPStreamMasqueradingAsCUDA(device).stream()", "nullptr"), ("_la_host", "_cpu_host")]
WORKER = """
import ctypes, sys, threading, torch
sys.path.insert(0, sys.argv[1])
import _cpu_host as h
stub = ctypes.CDLL(sys.argv[1] + "/stub.so")
h.bind(sys.argv[1] + "/stub.so")
need, wait, entered = (ctypes.c_size_t.in_dll(stub, q) for q in ("stub_need", "stub_wait", "stub_entered"))
A, y, x = torch.eye(4).repeat(2, 1, 1), torch.ones(2, 4), torch.ones(3)
calls = [lambda: h.potrf(A, True), lambda: h.potrf_backward(A, A, True), lambda: h.tri(True, A, A, True, False, False, 1.0),
         lambda: h.tri_backward(True, A, A, A, True, False, False, 1.0), lambda: h.syrk(A, False, 1.0), lambda: h.syrk_backward(A, A, False, 1.0),
         lambda: h.gemm2(A, A, False, False, 1.0), lambda: h.gemm2_backward(A, A, A, False, False, 1.0), lambda: h.potri(A, True),
         lambda: h.potri_backward(A, A, A, True), lambda: h.sumlogdiag(A), lambda: h.gp_criterion(A, y)]
every = lambda: [c() for c in calls]
what = sys.argv[2]
assert None not in every()
if what == "memory":
    small, (A, y), need.value = (A, y), (torch.eye(5).repeat(2, 1, 1), torch.ones(2, 5)), 1 << 60
    assert [r is None for r in every()] == [q != 10 for q in range(12)]  # (sumlogdiag takes no workspace)
    (A, y), need.value = small, 0  # (the answers for other sizes are remembered)
elif what == "threads":  # a thread goes on while another is in the library
    wait.value = 1
    t = threading.Thread(target=calls[0])
    t.start()
    while not entered.value:
        pass
    wait.value = 0
    t.join()
else:
    seen = []
    def f(v):
        seen.extend(every())
        return v.sum()
    F = torch.func
    {"grad": lambda: F.grad(f)(x), "jvp": lambda: F.jvp(f, (x,), (x,)), "jacrev": lambda: F.jacrev(f)(x), "hessian": lambda: F.hessian(f)(x),
     "vmap": lambda: F.vmap(f)(x[:, None]), "functionalize": lambda: F.functionalize(f)(x)}[what]()
    assert seen and set(seen) == {None}
assert None not in every()
print("done")
"""


@pytest.fixture(scope="module")
def cpu_host(tmp_path_factory):
    if shutil.which("g++") is None or shutil.which("gcc") is None:
        pytest.skip("no compiler")
    tmp = str(tmp_path_factory.mktemp("host"))
    with open(os.path.join(build.CSRC, "host_call.cpp")) as f:
        src = f.read()
    for a, b in CPU:
        assert a in src
        src = src.replace(a, b)
    with open(os.path.join(tmp, "host.cpp"), "w") as f:
        f.write(src)
    stub = "typedef unsigned long size_t;\nvolatile size_t stub_need, stub_wait, stub_entered;\n"
    for name in re.findall(r"LA_BIND\(\w+, (la_\w+)\)", src):
        stub += f"size_t {name}() {{ return stub_need; }}\n" if name.endswith("bytes") else f"int {name}() {{ stub_entered = 1; while (stub_wait); return 0; }}\n"
    with open(os.path.join(tmp, "stub.c"), "w") as f:
        f.write(stub)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", tmp + "/stub.so", tmp + "/stub.c"], check=True)
    subprocess.run([x if x != "-O2" else "-O0" for x in build.host_command(tmp + "/host.cpp", tmp + "/_cpu_host.so")], check=True)
    return tmp


@pytest.mark.parametrize("what", ["grad", "jvp", "jacrev", "hessian", "vmap", "functionalize", "memory", "threads"])
def test_calls_that_are_not_plain_end_in_none(cpu_host, what):
    r = subprocess.run([sys.executable, "-c", WORKER, cpu_host, what], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "done" in r.stdout, (r.returncode, r.stderr[-2000:])
