"""Builds libslowmo.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslowmo.so")
SOURCES = ["slowmo_kernels.hip", "slowmo_api.cpp", "slowmo_plan.cpp"]
HEADERS = ["slowmo_kernels.h", "slowmo_plan.h", os.path.join("..", "..", "include", "slowmo.h")]

# -ffp-contract=off: every product and sum rounds on its own, in source order
# (the order of the paper's formulas); the packed-fp32 feature is disabled.
# Kernel-argument preload: the first 14 words of a kernel's arguments are in its scalar registers when a
# wave starts, one trip to memory less in front of its first load (short lists: a step of 4.9 us 0.2-0.3
# us less, 0.95-0.97 of a round; long lists 0.99-1.00).  The words that lead to a wave's data come first.
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wextra",
         "-Wno-unused-parameter", "-mllvm", "-amdgpu-kernarg-preload-count=14"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES + HEADERS] + [os.path.abspath(__file__)]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not stale():
        return LIB
    cmd = [hipcc(), *FLAGS, "-x", "hip", *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the device-only target feature; that warning is expected
    err = "\n".join(ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stderr)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
