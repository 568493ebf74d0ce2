"""Build libsmcx.so in-tree with hipcc for gfx950.

Usage: python -m paper_2503_12591_amd.build   (or call build()).
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
LIB = os.path.join(PKG, "libsmcx.so")

SOURCES = ["smcx_kernels.hip", "smcx_coop.hip", "smcx_counts.hip", "smcx_qsro.hip", "smcx_sites.hip", "smcx_api.cpp"]

# -ffp-contract=off: every binary64 multiply and add of dE is rounded on its
# own, in the order written, so that trajectories are reproducible bit for bit.
# -packed-fp32-ops: packed FP32 instructions are kept out of the generated code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall",
         "-Wno-unused-command-line-argument"]


def build(verbose: bool = False) -> str:
    """Compile every source side by side, then link."""
    with tempfile.TemporaryDirectory() as tmp:
        jobs, objs = [], []
        for s in SOURCES:
            obj = os.path.join(tmp, s + ".o")
            cmd = ["hipcc"] + FLAGS + ["-I", INCLUDE, "-I", CSRC, "-c", os.path.join(CSRC, s), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            log = open(obj + ".log", "w+")
            jobs.append((subprocess.Popen(cmd, stdout=log, stderr=log), log))
            objs.append(obj)
        failed = False
        for p, log in jobs:
            if p.wait() != 0:
                log.seek(0)
                sys.stderr.write(log.read())
                failed = True
            log.close()
        if failed:
            raise RuntimeError("hipcc failed building libsmcx.so")
        link = ["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB + ".tmp"] + objs
        res = subprocess.run(link, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed linking libsmcx.so")
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
