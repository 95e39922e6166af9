"""Build libconvfirst.so (the gfx950 HIP kernels and the C ABI) in-tree.

    python -m paper_2404_03617_amd.build        # or build() from Python

Each csrc/*.hip file is compiled by hipcc for gfx950 into _build/, in
parallel, then linked into paper_2404_03617_amd/_lib/libconvfirst.so.  The
binding's argument checks (csrc/host/cf_args.cpp, host code against torch's
headers) become the CPython module _lib/_cf_args.so.
"""
from __future__ import annotations

import concurrent.futures as cfut
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB_DIR = os.path.join(PKG, "_lib")
LIB = os.path.join(LIB_DIR, "libconvfirst.so")
ARGS_SRC = os.path.join(CSRC, "host", "cf_args.cpp")
ARGS_LIB = os.path.join(LIB_DIR, "_cf_args.so")

ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed fp32 instructions are switched off for every kernel (the hardware
# forms v_pk_fma_f32 & co. are avoided on this target).
COMMON = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-I", INCLUDE, "-I", CSRC]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC] + COMMON + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), r.stderr[-8000:]))
    return obj


def build_args() -> str:
    """Compile the native argument checks; returns the module's path."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths

    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = ARGS_LIB + ".tmp"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), ARGS_SRC, "-o", tmp]
    for d in include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    cmd += ["-L" + tlib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath," + tlib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compiling %s failed:\n%s\n%s" % (ARGS_SRC, " ".join(cmd), r.stderr[-8000:]))
    os.replace(tmp, ARGS_LIB)
    return ARGS_LIB


def build(jobs: int | None = None) -> str:
    """Compile every kernel source and link the shared library, and the native
    argument checks; returns the library's path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    os.makedirs(LIB_DIR, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(len(srcs), max(1, (os.cpu_count() or 4)))
    with cfut.ThreadPoolExecutor(jobs) as ex:
        args = ex.submit(build_args)
        objs = list(ex.map(_compile, srcs))
        args.result()
    tmp = LIB + ".tmp"
    # hipBLASLt: the two GEMMs of the wide-block path (cf_libgemm.hip)
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC"] + objs + ["-L/opt/rocm/lib", "-lhipblaslt",
                                                                          "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), r.stderr[-8000:]))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
    sys.exit(0)
