"""What a call does on workspaces of other sizes than la_workspace_bytes names, without a GPU: the library runs in a process of its own
in which the HIP calls of the launch path are replaced by ones that only count the launches."""
import json
import os
import shutil
import subprocess
import sys

import pytest

SHIM = """
long la_launches;
int hipLaunchKernel(const void *f) { ++la_launches; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)(1ul << 50); return 0; }
int __hipPushCallConfiguration(void) { return 0; }
int __hipPopCallConfiguration(void *a, void *b, void *c, void *d) { return 0; }
"""

# [op, dt, batch, n, m, k, flags, bytes] -> [status, launches]; bytes null: -> what la_workspace_bytes answers; op 30, potrf on the library's own
# scratch array: the message as well
WORKER = """
import ctypes, json, sys
from ctypes import c_double as d, c_int as i, c_int64 as I, c_size_t as sz, c_void_p as vp
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
launches = ctypes.c_long.in_dll(shim, "la_launches")
for f in (lib.la_workspace_bytes, lib.la_gp_workspace_bytes, lib.la_sgp_workspace_bytes):
    f.restype = sz
lib.la_last_error.restype = ctypes.c_char_p
p = [vp((q + 1) << 44) for q in range(10)]  # operands, far apart and never dereferenced

def call(op, dt, batch, n, m, k, flags, w):
    if w is None:
        if op == 20:
            return lib.la_gp_workspace_bytes(i(dt), I(batch), i(n))
        if op == 21:
            return lib.la_sgp_workspace_bytes(i(dt), i(n), i(m))
        return lib.la_workspace_bytes(i(op), i(dt), I(batch), i(n), i(m), i(k))
    lower, trans, right = map(i, flags)
    b, n, m, k, dt = I(batch), i(n), i(m), i(k), i(dt)
    ws = (vp(1 << 50 if w else 0), sz(w), vp(0))
    before = launches.value
    tri = (dt, lower, trans, right, d(1), b, n, m)
    s = {
        0: lambda: lib.la_potrf_batched_ws(dt, lower, b, n, p[0], p[1], vp(0), *ws),
        1: lambda: lib.la_potrf_backward_ws(dt, lower, b, n, p[0], p[1], p[2], *ws),
        2: lambda: lib.la_trsm_batched_ws(*tri, p[0], p[1], p[2], *ws),
        3: lambda: lib.la_trmm_batched_ws(*tri, p[0], p[1], p[1], *ws),
        4: lambda: lib.la_syrk_batched_ws(dt, trans, d(1), b, n, k, p[0], p[1], *ws),
        5: lambda: lib.la_gemm2_batched_ws(dt, trans, right, d(1), b, m, n, k, p[0], p[1], p[2], *ws),
        6: lambda: lib.la_trsm_backward_ws(*tri, *p[:5], *ws),
        7: lambda: lib.la_trmm_backward_ws(*tri, *p[:5], *ws),
        8: lambda: lib.la_syrk_backward_ws(dt, trans, d(1), b, n, k, p[0], p[1], p[2], *ws),
        10: lambda: lib.la_potri_ws(dt, lower, b, n, p[0], p[1], *ws),
        11: lambda: lib.la_potri_backward_ws(dt, lower, b, n, p[0], p[1], p[2], p[3], *ws),
        20: lambda: lib.la_gp_criterion(dt, b, n, p[0], p[1], p[2], p[3], vp(0), *ws),
        21: lambda: lib.la_sgp_criterion(dt, n, m, *p[:4], d(1), *p[4:], *ws),
        30: lambda: lib.la_potrf_batched_noalloc(dt, lower, b, n, p[0], p[1], vp(0), vp(0)),
    }[op]()
    return [s, launches.value - before] + ([lib.la_last_error().decode()] if op == 30 and s else [])

print(json.dumps([call(*q) for q in json.load(sys.stdin)]))
"""

POTRF, BACKWARD, TRSM, TRMM, SYRK, GEMM2, TRSM_B, TRMM_B, SYRK_B, POTRI, POTRI_B = 0, 1, 2, 3, 4, 5, 6, 7, 8, 10, 11
GP, SGP, NOALLOC = 20, 21, 30
OPS = (POTRF, BACKWARD, TRSM, TRMM, SYRK, GEMM2, TRSM_B, TRMM_B, SYRK_B, POTRI, POTRI_B)
OK, WORKSPACE = 0, 4


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    from paper_1710_08717_amd import binding, build

    if not os.path.exists(binding.lib_path()):
        build.build(force=False)
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no C compiler")
    tmp = tmp_path_factory.mktemp("shim")
    (tmp / "shim.c").write_text(SHIM)
    subprocess.run([cc, "-shared", "-fPIC", "-w", "-o", str(tmp / "shim.so"), str(tmp / "shim.c")], check=True)

    def run(queries):
        r = subprocess.run([sys.executable, "-c", WORKER, str(tmp / "shim.so"), binding.lib_path()], input=json.dumps(queries),
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)

    return run


def test_more_workspace_is_never_refused_and_a_refused_call_launches_nothing(ask):
    """in steps of a sixteenth of what la_workspace_bytes names, among them products whose long inner dimension is split beside G + G^T"""
    sizes = [(1, 2048, 256, 256), (1, 4096, 128, 128), (2, 2048, 256, 128), (1, 2050, 256, 256), (1, 512, 64, 64), (128, 512, 64, 64),
             (4, 1024, 64, 64), (3, 700, 24, 24), (100, 200, 200, 200), (20, 51, 51, 51), (1, 129, 4099, 4099), (1, 64, 64, 4096)]
    cases = [(op, dt, *s, fl) for op in OPS for dt in (0, 1) for s in sizes for fl in ((1, 0, 0), (0, 1, 1))]
    full = ask([[*c, None] for c in cases])
    steps = [[w * q // 16 // 256 * 256 for q in range(17)] for w in full]
    got = iter(ask([[*c, w] for c, ws in zip(cases, steps) for w in ws]))
    wrong = []
    for c, ws in zip(cases, steps):
        accepted = False
        for w in ws:
            status, launches = next(got)
            if status not in (OK, WORKSPACE) or (status == WORKSPACE and (launches or accepted)) or (status == OK and not launches):
                wrong.append((c, w, status, launches))
            accepted = accepted or status == OK
        if not accepted:
            wrong.append((c, "the full size"))
    assert wrong == []


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("n", [129, 213, 214, 222, 300, 400, 512, 600, 1024, 1183, 2048, 3001])
def test_gradient_of_the_factorisation_runs_smaller_batches_on_a_larger_ones_workspace(ask, n, dt):
    """across the batches at which its block columns get narrower (128 | 129 among them) and its two forms change places"""
    batches = [b for b in (1, 2, 3, 4, 5, 8, 12, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 150, 256, 300, 600) if b * n * n < 2e8]
    full = ask([[BACKWARD, dt, b, n, 0, 0, (1, 0, 0), None] for b in batches])
    pairs = [(b, w, big) for w, big in zip(full, batches) for b in batches if b <= big]
    got = ask([[BACKWARD, dt, b, n, 0, 0, (1, 0, 0), w] for b, w, _ in pairs])
    assert [(b, big) for (b, w, big), (status, _) in zip(pairs, got) if status != OK] == []


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("op", [TRSM, TRMM, TRSM_B, TRMM_B, POTRI_B])
def test_matrices_of_33_to_64_rows_run_smaller_batches_on_a_larger_ones_workspace(ask, op, dt):
    """across the 1024 matrices from which one wavefront each does the operator without scratch"""
    batches = (1, 5, 100, 1000, 1024, 1025, 1536, 1537, 3072, 3073, 5000)
    for n, m in ((33, 49), (40, 60), (48, 80), (51, 51), (64, 100), (64, 300), (37, 700), (48, 2048), (64, 4096)):
        full = ask([[op, dt, b, n, m, 0, (1, 0, 0), None] for b in batches])
        queries = [[op, dt, b, n, m, 0, fl, w] for w, big in zip(full, batches) for b in batches if b <= big for fl in ((1, 0, 0), (0, 1, 1))]
        assert [q for q, (status, _) in zip(queries, ask(queries)) if status != OK] == []


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("op", [TRSM, TRSM_B])
def test_solves_of_17_to_32_rows_run_smaller_batches_on_a_larger_ones_workspace(ask, op, dt):
    """across the 3072 matrices from which one wavefront each takes more than 128 vectors without scratch"""
    batches = (1, 5, 1000, 3071, 3072, 3073, 5000)
    for n, m in ((17, 130), (20, 129), (24, 200), (31, 128), (32, 700), (24, 4096)):
        full = ask([[op, dt, b, n, m, 0, (1, 0, 0), None] for b in batches])
        queries = [[op, dt, b, n, m, 0, fl, w] for w, big in zip(full, batches) for b in batches if b <= big for fl in ((1, 0, 0), (0, 1, 1))]
        assert [q for q, (status, _) in zip(queries, ask(queries)) if status != OK] == []


@pytest.mark.parametrize("dt", [0, 1])
@pytest.mark.parametrize("op,batch,n", [(POTRF, 1, 801), (POTRF, 2, 961), (POTRF, 2, 1001), (POTRF, 1, 2001), (POTRF, 30, 901), (POTRF, 1, 6301),
                                        (BACKWARD, 1, 131), (BACKWARD, 3, 333), (BACKWARD, 1, 507), (BACKWARD, 100, 201), (BACKWARD, 1, 2501),
                                        (BACKWARD, 1, 6301), (POTRI, 1, 801), (GP, 1, 801), (GP, 2, 1001), (SGP, 1, 801), (SGP, 1, 1001)])
def test_odd_sizes_take_padded_copies_only_where_all_of_them_fit(ask, op, batch, n, dt):
    """a few steps of 256 bytes on both sides of every whole number of squares, rows padded or not, beside what the call has taken in any case"""
    es = 8 if dt else 4
    ld = (n * es + 15) // 16 * 16 // es
    case = [op, dt, batch, n, 2 * n if op == SGP else 0, 0, (1, 0, 0)]
    full, = ask([[*case, None]])
    fixed = {GP: (2 * n * n + 2 * n) * batch * es, SGP: (4 * n * n + 2 * n * n + 3 * n + 16) * es + 8}.get(op, 0)
    sizes = {full + 256 * q for q in range(-8, 2)}
    for squares in range(9):
        for row in (n, ld):
            at = (fixed + squares * batch * n * row * es) // 256 * 256
            sizes |= {at + 256 * q for q in range(-4, 60 if op == SGP else 12)}
    sizes = sorted(w for w in sizes if 0 <= w <= full + 256)
    got = ask([[*case, w] for w in sizes])
    states = [s for s, _ in got]
    assert set(states) <= {OK, WORKSPACE} and states == sorted(states, reverse=True) and states[sizes.index(full)] == OK
    assert [w for w, (s, launches) in zip(sizes, got) if (s == OK) != (launches > 0)] == []


@pytest.mark.parametrize("dt,op,batch,n,squares", [(1, POTRF, 1, 80001, 3), (1, POTRF, 1, 32769, 3), (0, POTRF, 1, 46341, 3), (1, POTRF, 40, 9001, 3),
                                                   (1, BACKWARD, 1, 80001, 0), (0, BACKWARD, 1, 46341, 0), (1, BACKWARD, 200000, 201, 2)])
def test_padded_copies_of_very_large_problems_are_not_counted(ask, dt, op, batch, n, squares):
    """what fits on the card without them still fits (288 GB; potrf of 80001 rows: operands 102, workspace 154)"""
    es = 8 if dt else 4
    full, = ask([[op, dt, batch, n, 0, 0, (1, 0, 0), None]])
    assert full <= squares * batch * n * n * es + (0 if squares else 1300 * n * es) + (64 << 20)


@pytest.mark.parametrize("dt,op,batch,n,squares", [(1, POTRF, 1, 32767, 4), (0, POTRF, 1, 46337, 4), (1, BACKWARD, 1, 32767, 2), (1, BACKWARD, 20000, 201, 3)])
def test_padded_copies_of_large_problems_are_counted(ask, dt, op, batch, n, squares):
    full, = ask([[op, dt, batch, n, 0, 0, (1, 0, 0), None]])
    assert full >= squares * batch * n * n * (8 if dt else 4)


@pytest.mark.parametrize("dt,batch,n,fits", [(1, 1, 2048, True), (1, 1, 2049, False), (1, 1, 1673, True), (1, 1, 1999, True), (1, 1, 2047, True),
                                             (1, 4, 1023, True), (1, 16, 512, True), (1, 17, 512, False), (0, 1, 2304, True), (0, 1, 2364, True),
                                             (0, 1, 2365, False), (0, 32, 512, True), (0, 33, 512, False), (1, 1000000, 64, True)])
def test_potrf_on_the_librarys_own_array_takes_what_fits_without_optional_room(ask, dt, batch, n, fits):
    """the limits that include/la.h states, and the size that a refusal names: with a workspace of that size the call runs, with less it does not"""
    for flags in ((1, 0, 0), (0, 0, 0)):
        (status, launches, *text), = ask([[NOALLOC, dt, batch, n, 0, 0, flags, 0]])
        assert (status, launches > 0) == ((OK, True) if fits else (WORKSPACE, False))
        if not fits:
            need = int(text[0].split("needs ")[1].split()[0])
            assert need > 64 << 20
            assert [s for s, _ in ask([[POTRF, dt, batch, n, 0, 0, flags, w] for w in (need, need - 256)])] == [OK, WORKSPACE]
