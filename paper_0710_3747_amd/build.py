"""Builds the HIP library libspinqp.so for gfx950 (in-tree, under _build/).

    python -m paper_0710_3747_amd.build

All HIP code is compiled with packed FP32 instructions disabled.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(OUT_DIR, "libspinqp.so")
# kernels.hip is compiled once per part (template families), in parallel
KERNEL_PARTS = 8
SOURCES = [f"kernels.hip:{n}" for n in range(KERNEL_PARTS)] + [
    "noalloc.hip", "planner.cpp", "abi.cpp", "batch.cpp", "autotune.cpp", "ensemble.cpp"]
ARCH = os.environ.get("SPINQP_ARCH", "gfx950")

HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
             "-mllvm", "-structurizecfg-skip-uniform-regions=true",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-function"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    os.makedirs(OUT_DIR, exist_ok=True)
    objs = []
    procs = []
    for entry in SOURCES:
        src, _, part = entry.partition(":")
        obj = os.path.join(OUT_DIR, os.path.splitext(src)[0] + (f"_{part}" if part else "") + ".o")
        if src.endswith(".hip"):
            defs = [f"-DSPIN_PART={part}"] if part else []
            cmd = [hipcc(), *HIP_FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
        else:   # host-only C++ (HIP runtime API, no device code)
            cmd = [hipcc(), "-O2", "-std=c++17", "-fPIC", "-Wall", "-c", os.path.join(CSRC, src),
                   "-o", obj]
        procs.append((src, cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                                                 text=True)))
        objs.append(obj)
    for src, cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and
                        "target-feature" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"compiling {src} failed:\n{' '.join(cmd)}\n{out}")
        if verbose and out.strip():
            print(out)
    tmp = LIB + ".tmp"
    subprocess.check_call([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
