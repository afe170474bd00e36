"""Builds the HIP library in-tree for gfx950:  python -m paper_2605_13907_amd.build"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libais_gfx950.so")
FAST = os.path.join(PKG, "_ais_fast.so")
SOURCES = ("api.hip", "sweeps.hip", "reductions.hip", "fp8.hip", "fp8_rows.hip", "fp8_table.hip", "fused.hip", "lm_head.hip",
           "lm_grad_gemm.hip")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-result",
    # packed-fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def fast_binding_command():
    """The binding's native calls: host code, against the torch that is installed.  -> (command, None), or (None, what is
    missing for them)."""
    try:
        from torch.utils import cpp_extension

        from paper_2605_13907_amd.binding import fast_stamp
    except ImportError as e:
        return None, f"torch ({e})"
    cxx = os.environ.get("CXX", "g++")
    if shutil.which(cxx) is None:
        return None, f"a host compiler ({cxx})"
    python_headers = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(python_headers, "Python.h")):
        return None, f"Python.h (in {python_headers})"
    dirs = [*cpp_extension.include_paths(), python_headers, os.path.join(ROOT, "include")]
    return [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f'-DAIS_FAST_STAMP="{fast_stamp()}"',
            *[f"-I{d}" for d in dirs], os.path.join(CSRC, "fast_binding.cpp"), "-o", FAST,
            *[f"-L{d}" for d in cpp_extension.library_paths()], "-ltorch_python", "-ltorch_cpu", "-lc10"], None


def build(verbose: bool = True) -> str:
    """Compiles the library, which needs hipcc alone, and beside it the binding's native calls where there is what they need.
    Neither is left over from an earlier build if this one fails."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    fast, missing = fast_binding_command()
    for built in (LIB, FAST):
        if os.path.exists(built):
            os.remove(built)
    if verbose:
        print(" ".join(cmd), flush=True)
        print(" ".join(fast) if fast else f"the binding's native calls are not built: no {missing}", flush=True)
    beside = subprocess.Popen(fast) if fast else None
    try:
        subprocess.run(cmd, check=True)
    finally:
        rc = beside.wait() if beside else 0
    if rc != 0:
        raise subprocess.CalledProcessError(rc, fast)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
