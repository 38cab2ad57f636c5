"""Build libsbi.so (gfx950) in-tree with hipcc.

Usage: python -m paper_2310_19840_amd.build [--jobs N]
"""
from __future__ import annotations

import argparse
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libsbi.so")
BUILD = os.path.join(HERE, "_build")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
ARCH = os.environ.get("SBI_OFFLOAD_ARCH", "gfx950")
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from emitting packed FP32 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

UNITS = [
    ("sbi_kernels.hip", "sbi_k64.o", ["-DSBI_REAL=double"]),
    ("sbi_kernels.hip", "sbi_k32.o", ["-DSBI_REAL=float"]),
    ("sbi_full.hip", "sbi_full64.o", ["-DSBI_REAL=double"]),
    ("sbi_full.hip", "sbi_full32.o", ["-DSBI_REAL=float"]),
    ("sbi_line.hip", "sbi_line64.o", ["-DSBI_REAL=double", "-DSBI_LINE_MAIN"]),
    ("sbi_line.hip", "sbi_line32.o", ["-DSBI_REAL=float"]),
    ("sbi_dispatch.hip", "sbi_dispatch.o", []),
    ("sbi_api.hip", "sbi_api.o", []),
    ("sbi_net.hip", "sbi_net.o", []),
    ("sbi_net_api.hip", "sbi_net_api.o", []),
]


def _compile(unit):
    src, obj, extra = unit
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", os.path.join(BUILD, obj)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(jobs: int = 4, verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        objs = list(ex.map(_compile, UNITS))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp,
           *[os.path.join(BUILD, o) for o in objs]]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=4)
    a = ap.parse_args()
    build(a.jobs, verbose=True)
    sys.exit(0)
