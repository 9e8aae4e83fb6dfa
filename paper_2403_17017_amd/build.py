"""Builds libseer.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libseer.so")
SOURCES = ["seer_api.hip", "spmv_rowmapped.hip", "spmv_mergepath.hip", "spmv_workoriented.hip", "spmv_adaptive.hip", "spmv_ell.hip", "spmv_coo.hip", "spmv_slab.hip", "spmv_bins.hip", "spmv_long.hip", "features.hip", "spmv_auto.hip"]
FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-fno-gpu-rdc",
    # the compiler must not form packed-fp32 instructions on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


MARSHAL = os.path.join(HERE, "_marshal.so")    # the binding's argument marshalling (host code only)


def build_marshal(verbose: bool = False) -> str:
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"],
           "-o", MARSHAL, os.path.join(CSRC, "marshal.c")]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    return MARSHAL


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    build_marshal(verbose)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
