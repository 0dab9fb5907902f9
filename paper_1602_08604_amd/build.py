"""Build the gfx950 HIP library (liblre.so) in-tree with hipcc.

Run ``python -m paper_1602_08604_amd.build`` (or __graft_entry__.build()).  The
library lands in paper_1602_08604_amd/_lib/ so that it travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB_DIR = os.path.join(PKG, "_lib")
LIB = os.path.join(LIB_DIR, "liblre.so")
SOURCES = [os.path.join(PKG, "csrc", f)
           for f in ("lre_abi.hip", "lre_batch.hip", "lre_project.hip", "lre_membench.hip")]
DEPS = SOURCES + [os.path.join(PKG, "csrc", f) for f in ("lre_kernels.hpp", "lre_tile.hpp", "lre_povm.hpp", "lre_internal.hpp")] + [
    os.path.join(ROOT, "include", "lre.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # Packed FP32 instructions stay off (compiler-generated v_pk_*_f32 are avoided).
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"),
]


def build(force: bool = True, verbose: bool = False) -> str:
    os.makedirs(LIB_DIR, exist_ok=True)
    if not force and os.path.exists(LIB) and all(
            os.path.getmtime(LIB) >= os.path.getmtime(d) for d in DEPS):
        return LIB
    tmp = LIB + ".tmp"
    cmd = [HIPCC, *FLAGS, *SOURCES, "-o", tmp, "-lrocsolver", "-lrocblas"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{err}")
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
