"""Builds libqeft.so for gfx950 with hipcc (cross-compiles without a GPU), and the host-side module between torch tensors and its calls.

    python -m paper_2410_08661_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libqeft.so")
MARSHAL_PATH = os.path.join(HERE, "_marshal.so")

SOURCES = ["api.hip", "generic.hip", "pack.hip", "irregular.hip", "reorder.hip", "gemv.hip", "gemv_dot.hip", "gemm.hip", "gemm_mid.hip", "gemm_tile.hip", "dx_panel.hip", "noalloc.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept off for every device function of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# The quantizers take integer decisions from fp32 arithmetic that is specified operation by operation
# (one rounding each): no multiply-add fusion anywhere in that file, its inlined header functions included.
EXTRA_FLAGS = {"pack.hip": ["-ffp-contract=off"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    noise = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if noise:
        sys.stderr.write(noise + "\n")
    return obj


def _build_marshal() -> bool:
    """The binding does without it (calls then go through ctypes), so a machine that cannot build it gets the library all the same, and is told."""
    import torch
    if os.path.exists(MARSHAL_PATH):
        os.remove(MARSHAL_PATH)   # (one of an older source or torch may not stay)
    t = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(HIPCC))) if os.path.isabs(HIPCC) else "/opt/rocm"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(t, "include"), "-I", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-I", os.path.join(rocm, "include"), "-I", sysconfig.get_paths()["include"], os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL_PATH,
           "-L", os.path.join(t, "lib"), "-ltorch_python", "-lc10", "-lc10_hip"]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed = f"{r.stdout}\n{r.stderr}" if r.returncode != 0 else None
    except OSError as e:
        failed = str(e)
    if failed is not None:
        sys.stderr.write(f"marshal.cpp is not built, calls go through ctypes:\n{failed}\n")
    return failed is None


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        host = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, SOURCES))
        host.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    if verbose:
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build()
