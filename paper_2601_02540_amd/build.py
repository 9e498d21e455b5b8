"""Builds the gfx950 shared library ``libsgn.so`` in-tree with hipcc.

``python -m paper_2601_02540_amd.build`` compiles every HIP source of the
package.  The library links only against the HIP runtime; it has no PyTorch
dependency.
"""

from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libsgn.so")
SOURCES = [os.path.join(CSRC, f) for f in ("sgn_lib.hip", "sgn_batch.hip", "sgn_adjoint.hip", "sgn_relax.hip",
                                                "sgn_totals.hip", "sgn_noalloc.hip", "sgn_fsal.hip", "sgn_march.hip",
                                                "sgn_small.hip")]
HEADERS = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith((".hpp", ".h"))] + [
    os.path.join(INCLUDE, "sgn.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # No packed FP32 instructions in the gfx950 code.  The host pass warns that
    # it does not know the feature (it is an AMDGPU one); the device pass
    # applies it (tests/test_build_flags.py checks the built code objects).
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE,
    "-I", CSRC,
]


def build(verbose: bool = False) -> str:
    """Compiles every translation unit in parallel, then links the shared library."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    for p, cmd in procs:
        if p.wait() != 0:
            raise subprocess.CalledProcessError(p.returncode, cmd)
    link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.check_call(link)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
