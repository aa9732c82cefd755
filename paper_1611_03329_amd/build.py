"""Builds the gfx950 shared library ``liblbm.so`` (HIP kernels + C ABI) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
SRCS = [os.path.join(PKG, "csrc", f) for f in ("lbm_capi.hip", "lbm_multi.hip")]
LIB = os.path.join(PKG, "liblbm.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # fused multiply-adds only where one source expression has the form a * b + c:
    # the rounding of every step is then the same in every kernel variant
    # (check modes, batch or single lattice), whatever else the compiler sees
    "-ffp-contract=on",
    "-Wall", "-Wno-unused-function",
    # keep the compiler from forming packed-FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def build(extra_flags=(), verbose: bool = False) -> str:
    """Compiles the sources side by side and links the library."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as work:
        objs, jobs = [], []
        for src in SRCS:
            obj = os.path.join(work, os.path.basename(src) + ".o")
            cmd = [hipcc(), *HIPCC_FLAGS, *extra_flags, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            objs.append(obj)
            jobs.append((cmd, subprocess.Popen(cmd)))
        failed = [(job.returncode, cmd) for cmd, job in jobs if job.wait() != 0]
        if failed:
            raise subprocess.CalledProcessError(*failed[0])
        subprocess.run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *extra_flags, *objs, "-o", tmp], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(sys.argv[1:], verbose=True)
