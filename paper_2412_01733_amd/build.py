"""Build libtreecode.so (the HIP kernels and the C ABI) for gfx950, in-tree.

    python -m paper_2412_01733_amd.build

Every translation unit is compiled with hipcc for gfx950 only.  Flags:
  -ffp-contract=off   no implicit FMA contraction: the key quantisation and the
                      FP64 moments are bit-reproducible; the walk writes its
                      fused multiply-adds explicitly.
  -Xclang -target-feature -Xclang -packed-fp32-ops
                      no packed-FP32 instructions are generated.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libtreecode.so")
BUILD_DIR = os.path.join(os.path.dirname(HERE), "_build")

SOURCES = ["keys.hip", "scan.hip", "sort.hip", "sort_small.hip", "build.hip", "moments.hip", "order.hip", "walk.hip", "walk_forward.hip", "walk_adjoint.hip", "walk_split.hip", "walk_direct.hip", "adjoint.hip", "diag.hip",
           "integrate.hip", "capi.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), r.stderr))
    return obj


def build(verbose: bool = False) -> str:
    """Compile every HIP source and link libtreecode.so; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = OUT + ".tmp%d" % os.getpid()
    # -z defs: a symbol declared but defined nowhere fails the link, not the load
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-z,defs", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), r.stderr))
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
