"""Builds libumbir.so, the gfx950 HIP library behind include/umbir.h, in-tree.

    python -m paper_2202_09703_amd.build

Every HIP source is compiled with packed-FP32 instruction selection turned
off (the kernels are written for plain FP32 FMAs).
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libumbir.so")
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: install ROCm or set HIPCC")


def sources():
    return sorted(glob.glob(os.path.join(PKG, "csrc", "*.hip")))


def build(verbose: bool = False) -> str:
    """Compiles every source (side by side) into libumbir.so (always rebuilds); returns its path."""
    tmp = LIB + ".tmp"
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)

    with tempfile.TemporaryDirectory() as objs:
        pairs = [(s, os.path.join(objs, os.path.basename(s) + ".o")) for s in sources()]
        with ThreadPoolExecutor(max_workers=4) as pool:
            list(pool.map(lambda p: run([hipcc(), *flags, "-c", p[0], "-o", p[1]]), pairs))
        run([hipcc(), f"--offload-arch={ARCH}", "-fPIC", "-shared", *(o for _, o in pairs), "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
