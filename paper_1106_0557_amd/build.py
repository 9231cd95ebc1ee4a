"""Build ``libpspfft.so`` (HIP, gfx950) in-tree.

Usage: ``python -m paper_1106_0557_amd.build`` or ``build()`` from Python.
Every call recompiles (the build check compiles each time it is asked to).
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpspfft.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# Packed FP32 instructions are disabled for every HIP compile.  The sign of a
# zero plays no part in the results, so x + 0 folds to x (the known-zero halves
# of padded lines cost no additions).
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-parameter", "-fno-signed-zeros",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]

DEVICE_SOURCES = ([f"pass_{p}_e{e}.hip" for p in ("f32", "f64") for e in (36, 24, 20, 16)]
                  + [f"mix_{p}_{c}.hip" for p in ("f32", "f64") for c in "edcba"]
                  + ["mix_plane_f32.hip", "mix_plane_f64.hip", "line_generic.hip",
                     "mix_info.hip", "green.hip", "noalloc.hip"])
HOST_SOURCES = ["pspfft_runtime.cpp"]


def _run(cmd):
    print("+", " ".join(cmd), flush=True)
    subprocess.check_call(cmd)


def build(verbose: bool = True, jobs: int = 8) -> str:
    out_dir = tempfile.mkdtemp(prefix="pspfft_build_")
    # at most `jobs` compilers at a time (each takes one CPU), the longest first
    sources = DEVICE_SOURCES + HOST_SOURCES
    objs = [os.path.join(out_dir, src + ".o") for src in sources]
    cmds = [[HIPCC, f"--offload-arch={ARCH}", *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
            for src, obj in zip(sources, objs)]

    def compile_one(cmd):
        if verbose:
            print("+", " ".join(cmd), flush=True)
        return subprocess.call(cmd)

    with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
        for cmd, rc in zip(cmds, pool.map(compile_one, cmds)):
            if rc != 0:
                raise RuntimeError("compile failed: " + " ".join(cmd))
    tmp = LIB + ".tmp"
    _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    for o in objs:
        os.unlink(o)
    os.rmdir(out_dir)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
