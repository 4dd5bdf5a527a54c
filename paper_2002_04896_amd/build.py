"""Build the HIP library libcroft.so for gfx950 (in place, next to this file).

hipcc compiles every source of csrc/ for --offload-arch=gfx950; the objects go
to _build/ at the repository root and are linked into
paper_2002_04896_amd/libcroft.so.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libcroft.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["croft_entries_c64.hip", "croft_entries_c128.hip", "croft_entries_c16f.hip",
           "croft_entries_c16b.hip", "croft_group_c64.hip", "croft_group_c128.hip", "croft_group_c16f.hip",
           "croft_group_c16b.hip", "croft_group_c16f_x.hip", "croft_group_c16b_x.hip", "croft_group_conv.hip",
           "croft_kernels.hip", "croft_batch.hip", "croft_bluestein.hip", "croft_noalloc.hip", "croft_transpose.hip", "croft_plan.cpp", "croft_api.cpp",
           "croft_tune.cpp"]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", f"-I{INCLUDE}", f"-I{CSRC}"]
# the device code must not use packed FP32 instructions
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src + ".o")
    path = os.path.join(CSRC, src)
    # kernels: no implicit contraction (their fused multiply-adds are explicit)
    lang = ["-x", "hip", "-ffp-contract=off"] if src.endswith(".hip") else []
    cmd = [HIPCC, *COMMON, *DEVICE, *lang, "-c", path, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile and link libcroft.so; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
