"""Builds libcwac_hip.so (the C-ABI library) in-tree with hipcc for gfx950, and beside it the Python extension through which
the binding makes its most frequent calls."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libcwac_hip.so")

SOURCES = ["status.hip", "quantize.hip", "calib_stats.hip", "fold_epilogue.hip", "qlinear_forward.hip", "qlinear_fast.hip",
           "qlinear_splitk.hip", "probe.hip", "w4a16.hip", "block_glue.hip"]

# -ffp-contract=off: the epilogue and the fold are defined as sequences of single
# roundings; packed fp32 instructions are disabled for the device pass.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(src: str, extra=(), suffix: str = "") -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + suffix + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    subprocess.run(cmd, check=True, stderr=subprocess.PIPE, text=True)
    return obj


FAST_CALLS = os.path.join(PKG, "_fast_calls.so")


def _build_fast_calls() -> None:
    """csrc/fast_calls.cpp: host code only, against the headers of Python and of the installed torch."""
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
                    f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include"),
                    "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include/torch/csrc/api/include"),
                    "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
                    os.path.join(CSRC, "fast_calls.cpp"), "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
                    "-lc10_hip", "-o", FAST_CALLS], check=True, stderr=subprocess.PIPE, text=True)


def build_library(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    try:
        with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
            calls = ex.submit(_build_fast_calls)
            objs = list(ex.map(_compile, SOURCES))
            calls.result()
        subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB],
                       check=True, stderr=subprocess.PIPE, text=True)
    except subprocess.CalledProcessError as e:
        sys.stderr.write(e.stderr or "")
        raise
    if verbose:
        print(f"built {LIB}")
    return LIB


STAMP_LIB = os.path.join(PKG, "libcwac_hip_timeline.so")


def build_timeline_library(verbose: bool = True) -> str:
    """Development build for `bench.py --tile-timeline`: the same library with the forward kernels
    compiled with -DCWAC_V_STAMP, which makes every wavefront of the direct-to-LDS kernels record
    100 MHz time stamps at five points of each tile and exports cwac_debug_stamps to read them.
    Never loaded by the product path (binding.lib() loads libcwac_hip.so)."""
    build_library(verbose=False)
    try:
        obj = _compile("qlinear_fast.hip", extra=("-DCWAC_V_STAMP",), suffix="_timeline")
        others = [os.path.join(BUILD, os.path.splitext(f)[0] + ".o") for f in SOURCES if f != "qlinear_fast.hip"]
        subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *others, obj, "-o", STAMP_LIB],
                       check=True, stderr=subprocess.PIPE, text=True)
    except subprocess.CalledProcessError as e:
        sys.stderr.write(e.stderr or "")
        raise
    if verbose:
        print(f"built {STAMP_LIB}")
    return STAMP_LIB


if __name__ == "__main__":
    if "--timeline" in sys.argv[1:]:
        build_timeline_library()
    else:
        build_library()
