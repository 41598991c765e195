"""Build libmcb.so (gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmcb.so")
CEILING = os.path.join(HERE, "mcb_ceiling")  # standalone copy / plain-pull bandwidth probe
SOURCES = ["api.hip", "geometry.hip", "step2d.hip", "tile2d.hip", "step3d.hip", "flat3d.hip", "monitor.hip",
           "download.hip", "adjoint.hip", "adjoint2d.hip", "adjoint3d.hip"]
ARCH = os.environ.get("MCB_OFFLOAD_ARCH", "gfx950")

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed FP32 instructions are disabled for every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc, *[f for f in FLAGS if f != "-shared"], "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    cmd = [hipcc, *[f for f in FLAGS if f not in ("-shared", "-fPIC")], os.path.join(CSRC, "ceiling.hip"), "-o", CEILING + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(CEILING + ".tmp", CEILING)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
