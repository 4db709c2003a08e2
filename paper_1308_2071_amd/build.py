"""Build liblbmpm.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_1308_2071_amd.build          # build (always recompiles)
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "liblbmpm.so")
SOURCES = ["lbm_abi.cpp", "lbm_kernels.hip", "lbm_tile.hip", "lbm_adjoint.hip", "lbm_batch.hip"]
ARCH = os.environ.get("LBM_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
    # no packed FP32 instructions (v_pk_*_f32) anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no fused multiply-add contraction: every kernel rounds each operation as written, so the
    # batched, plain and adjoint kernels give bitwise-identical forward results
    "-ffp-contract=off", "-Wall", "-Wno-unused-result",
    "-I", INCLUDE, "-I", CSRC,
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    return compile_shared(srcs, LIB, verbose)


def compile_shared(srcs, out: str, verbose: bool = False) -> str:
    """A shared library from HIP sources with the library's own flags."""
    tmp = out + ".tmp"
    cmd = [hipcc()] + FLAGS + ["-o", tmp] + list(srcs)
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
