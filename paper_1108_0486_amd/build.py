"""Builds libxg.so (HIP for gfx950) in-tree with hipcc.

    python -m paper_1108_0486_amd.build
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(PKG, "libxg.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SOURCES = ["xg_kernels.hip", "xg_family.hip", "xg_split_tables.hip", "xg_plan_dev.hip", "xg_static.hip",
           "xg_util.hip", "xg_api.cpp", "xg_serve.cpp", "xg_jump.cpp", "xg_plan.cpp", "xg_tune.cpp"]

# -packed-fp32-ops: no packed FP32 instructions in generated code.
# -ffp-contract=off: every FP32 operation rounds as written (no implicit FMA).
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fvisibility=default",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def split_tables(folder: str, verbose: bool = False) -> None:
    """Writes folder/xg_split_tables.inc: the jump polynomials of xg_split.h,
    from the library's own jump code."""
    gen = os.path.join(folder, "split_tables_gen")
    cmd = [HIPCC, "-x", "c++", "-O2", "-std=c++17", "-I", INCLUDE, "-I", CSRC,
           os.path.join(CSRC, "split_tables_gen.cpp"), os.path.join(CSRC, "xg_jump.cpp"), "-o", gen]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    subprocess.run([gen, os.path.join(folder, "xg_split_tables.inc")], check=True)


def build(verbose: bool = False, out: str | None = None) -> str:
    target = out or LIB_PATH
    tmp = target + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as folder:
        split_tables(folder, verbose)
        cmd = [HIPCC, *FLAGS, "-I", INCLUDE, "-I", CSRC, "-I", folder,
               *[os.path.join(CSRC, s) for s in SOURCES], "-o", tmp]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    os.replace(tmp, target)
    return target


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
