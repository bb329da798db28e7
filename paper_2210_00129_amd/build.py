"""Builds libsbp.so (the C-ABI library) in-tree with hipcc for gfx950, and _native.so (part of the Python binding).

    python -m paper_2210_00129_amd.build

Cross-compiles without a GPU.  Packed-fp32 instructions are switched off for every
translation unit.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = ["sbp_api.hip", "sbp_sampler.hip", "sbp_gather.hip", "sbp_linear.hip", "sbp_linear_f32.hip", "sbp_dwconv.hip", "sbp_pointwise.hip", "sbp_attention.hip", "sbp_static.hip"]
LIB = os.path.join(HERE, "libsbp.so")
NATIVE = os.path.join(HERE, "_native.so")        # the binding of the calls of every step (host code, against torch's headers)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def build_native() -> subprocess.Popen:
    import torch
    t = os.path.dirname(torch.__file__)
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        raise RuntimeError("g++ not found")
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *["-I" + i for i in inc], os.path.join(HERE, "csrc", "sbp_binding.cpp"), "-o", NATIVE + ".tmp",
           "-L" + os.path.join(t, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python", "-Wl,-rpath," + os.path.join(t, "lib")]
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def build(verbose: bool = True) -> str:
    build_dir = os.path.join(ROOT, "_build")
    os.makedirs(build_dir, exist_ok=True)
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        cmd = [hipcc(), *HIPCC_FLAGS, *inc, "-c", os.path.join(HERE, "csrc", src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    native = build_native()
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    out, _ = native.communicate()
    if native.returncode != 0:
        raise RuntimeError("g++ failed on sbp_binding.cpp:\n" + out)
    os.replace(tmp, LIB)
    os.replace(NATIVE + ".tmp", NATIVE)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
