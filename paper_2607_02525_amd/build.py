"""Builds libpeek.so for gfx950 in-tree with hipcc, and beside it a variant for tests.

Usage: python paper_2607_02525_amd/build.py
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libpeek.so")
CALIB_LIB = os.path.join(HERE, "libpeek_calib.so")   # measurement helper for bench.py
# The same library with what a test cannot bring about otherwise: sampled places known
# beforehand, and waits between workgroups that give up at once
FORCED_LIB = os.path.join(HERE, "libpeek_forced.so")
FORCED = ["-DPEEK_SAMPLE_SEED=0", "-DPEEK_WAIT_SPINS=0"]
BUILD_DIR = os.path.join(HERE, "_build")

SOURCES = ["peek_host.hip", "peek_walk.hip", "peek_signals.hip", "peek_evict.hip", "peek_blocks.hip",
           "peek_noalloc.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-function",
    # gfx950 only; keep the compiler from forming packed fp32 ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + INCLUDE,
]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def _link(lib, objs, verbose):
    tmp = lib + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    objs, forced, jobs = [], [], []
    for src in SOURCES:
        for made, prefix, defines in ((objs, "", []), (forced, "forced_", FORCED)):
            obj = os.path.join(BUILD_DIR, prefix + src.replace(".hip", ".o"))
            made.append(obj)
            jobs.append([HIPCC, *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", obj])
    with ThreadPoolExecutor(4) as pool:
        list(pool.map(lambda cmd: _run(cmd, verbose), jobs))
    _link(LIB, objs, verbose)
    _link(FORCED_LIB, forced, verbose)
    tmp = CALIB_LIB + ".tmp"
    _run([HIPCC, *FLAGS, "-shared", "-o", tmp, os.path.join(CSRC, "peek_calib.hip")], verbose)
    os.replace(tmp, CALIB_LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
