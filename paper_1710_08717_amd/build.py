"""Compiles the HIP sources under ``csrc/`` into ``libla_mi355x.so`` (gfx950 only) and the binding's host part,
``csrc/host_call.cpp``, into ``_la_host.so``.

hipcc cross-compiles without a GPU, so this runs on the build host; the shared object
then travels with the tree to the GPU machine.  Run as ``python -m paper_1710_08717_amd.build``.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libla_mi355x.so")
HOST = os.path.join(PKG, "_la_host.so")

SOURCES = ["tiny.hip", "tiny_ops.hip", "tiny_rows.hip", "leaf.hip", "small_wave.hip", "trsm_stream.hip", "gemm.hip", "elem.hip", "kalman.hip", "la_api.hip"]
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-fno-gpu-rdc",
    # fuse multiply-adds only where the source says fma() or writes a*b+c in one expression:
    # cross-statement contraction would make mirrored entries of symmetric results differ by an ulp
    "-ffp-contract=on",
    "-Wall",
    "-Wno-unused-command-line-argument",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
    "-I", CSRC,
]


def _newer(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src):
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def host_command(src, out):
    """The compiler's call for the binding's host part."""
    import sysconfig

    import torch

    base = os.path.dirname(torch.__file__)
    inc = [os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
           "/opt/rocm/include", sysconfig.get_paths()["include"]]
    libs = ["torch_python", "torch_cpu", "torch_hip", "c10", "c10_hip"]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", *[x for d in inc for x in ("-isystem", d)],
            "-I", os.path.join(ROOT, "include"), src, "-o", out,
            "-L", os.path.join(base, "lib"), *[f"-l{x}" for x in libs]]  # (found by torch's own import, which comes first)


def _build_host():
    subprocess.check_call(host_command(os.path.join(CSRC, "host_call.cpp"), HOST))


def build(force=True, jobs=8):
    """Compile every HIP source and link the C-ABI library, and the binding's host part; returns the library's path."""
    os.makedirs(BUILD, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")] + [
        os.path.join(ROOT, "include", "la.h")
    ]
    todo = [
        s for s in SOURCES
        if force or _newer(os.path.join(BUILD, os.path.splitext(s)[0] + ".o"), [os.path.join(CSRC, s)] + headers)
    ]
    host = force or _newer(HOST, [os.path.join(CSRC, "host_call.cpp"), os.path.join(ROOT, "include", "la.h")])
    with ThreadPoolExecutor(max_workers=min(jobs, len(todo) + 1)) as ex:
        part = ex.submit(_build_host) if host else None
        list(ex.map(_compile, todo))
        if part:
            part.result()
    objs = [os.path.join(BUILD, os.path.splitext(s)[0] + ".o") for s in SOURCES]
    if todo or not os.path.exists(LIB):
        subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv))
