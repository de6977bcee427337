"""Build libbgk.so (HIP for gfx950) in-tree with hipcc.

Every HIP translation unit is compiled with packed-FP32 instructions turned
off, and with floating-point contraction limited to single source expressions
(-ffp-contract=on): which multiply-adds fuse is then fixed by the source, so
code that is inlined into several kernels (one stage work item in the
single-solver and the batched stage kernels) rounds identically in each. The
library lands next to this file and is what the binding loads.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libbgk.so")
OBJDIR = os.path.join(ROOT, "_build")
SOURCES = ["bgk_runtime.hip", "bgk_kernels.hip", "bgk_exchange.hip", "bgk_hexwalk.hip",
           "bgk_rows.hip", "bgk_xwalk.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=on",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed for {src}")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


def build_checks(only_missing: bool = False) -> str:
    """Library of device functions that a test calls directly (tests/*.hip)."""
    src = os.path.join(ROOT, "tests", "bf16_pair_check.hip")
    lib = os.path.join(ROOT, "tests", "libbf16pair.so")
    if not (only_missing and os.path.exists(lib)):
        tmp = lib + ".tmp"
        r = subprocess.run([HIPCC, *FLAGS, "-shared", src, "-o", tmp], capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError(f"hipcc failed for {src}")
        os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    build()
    build_checks()
