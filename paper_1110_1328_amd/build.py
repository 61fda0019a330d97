"""Build libbayeslsh.so for gfx950 with hipcc (in-tree).

    python -m paper_1110_1328_amd.build

Each source compiles to an object under paper_1110_1328_amd/_build/ (in
parallel), then the objects link into paper_1110_1328_amd/libbayeslsh.so.
build_bounds() builds tests/native/libbounds.so, the kernels that measure the
hardware's functions for test_gpu_bounds.py.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbayeslsh.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
SOURCES = ["api.hip", "verify.hip", "sigs.hip", "batched.hip", "banding.hip", "serving.hip", "tables.cpp", "server.cpp"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-I", os.path.join(HERE, "..", "include")]
# hipcc-only: no packed FP32 instructions in device code
DEVICE = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-fno-gpu-flush-denormals-to-zero"]


def _compile(src: str) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(BUILD, src + ".o")
    if src.endswith(".hip"):
        cmd = [HIPCC, "-x", "hip"] + COMMON + DEVICE + ["-c", path, "-o", obj]
    else:   # host-only C++ (HIP runtime API calls, no kernels)
        cmd = [HIPCC] + COMMON + ["-D__HIP_PLATFORM_AMD__", "-pthread", "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-pthread", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr))
    os.replace(tmp, LIB)
    if verbose:
        print(LIB)
    return LIB


def build_bounds(verbose: bool = False) -> str:
    native = os.path.join(HERE, "..", "tests", "native")
    out = os.path.join(native, "libbounds.so")
    tmp = out + ".tmp%d" % os.getpid()
    cmd = [HIPCC, "-x", "hip"] + COMMON + DEVICE + ["-shared", os.path.join(native, "bounds.hip"), "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("build failed: %s\n%s\n%s" % (" ".join(cmd), r.stdout, r.stderr))
    os.replace(tmp, out)
    if verbose:
        print(out)
    return out


if __name__ == "__main__":
    build(verbose=True)
    build_bounds(verbose=True)
    sys.exit(0)
