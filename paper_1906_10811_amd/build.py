"""Ahead-of-time build of libfd.so for gfx950 (hipcc), in-tree.

    python -m paper_1906_10811_amd.build

Kernels are compiled with packed-FP32 instructions disabled; the host
translation units are ordinary C++ linked against the HIP runtime.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libfd.so")
ARCH = "gfx950"

# the 3D step's instantiations are spread over units of similar size that
# compile in parallel (the longest first)
HIP_SOURCES = ["fd_step3d_f16_diff.hip", "fd_step3d_bf16_diff.hip", "fd_step3d_f32.hip",
               "fd_step3d_f16.hip", "fd_step3d_bf16.hip", "fd_step3d_f16_cached.hip", "fd_step3d_bf16_cached.hip",
               "fd_diffuse2d.hip", "fd_step2d.hip", "fd_kernels.hip"]
HOST_SOURCES = ["fd_api.cpp", "fd_serve.cpp", "fd_diffusion.cpp", "fd_checkpoint.cpp"]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "-I" + os.path.join(ROOT, "include")]
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for c in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("build failed: %s\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr))
    return r


def build(verbose: bool = False) -> str:
    hipcc = _hipcc()
    os.makedirs(BUILD, exist_ok=True)
    jobs = []
    objs = []
    for src in HIP_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        jobs.append([hipcc] + COMMON + DEVICE + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    for src in HOST_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        # host-only translation units: no device pass
        jobs.append([hipcc] + COMMON + ["-x", "hip", "--cuda-host-only", "--offload-arch=" + ARCH, "-c",
                                        os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1, len(jobs))) as ex:
        for r in ex.map(_run, jobs):
            if verbose and r.stderr:
                print(r.stderr, file=sys.stderr)
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([hipcc, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + objs + ["-lpthread"])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
