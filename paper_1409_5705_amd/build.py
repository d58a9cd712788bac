"""Builds libsfb.so (HIP, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsfb.so")
PEAKS = os.path.join(HERE, "sfb_peaks")
SOURCES = ["sfb_api.hip", "gemm_f32.hip", "gemm_f32x3.hip", "gemm_bf16.hip", "apply_gather.hip", "forward_bf16.hip", "rowops.hip", "sparse.hip", "ssp.cpp"]
FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are not trusted on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950 and link the shared library."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        if verbose and r.stderr.strip():
            print(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=min(4, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(tmp, LIB)
    # the stand-alone MFMA / HBM probe behind `bench.py --peaks`
    tmp = PEAKS + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc] + FLAGS + ["-o", tmp, os.path.join(CSRC, "peaks.hip")], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for peaks.hip:\n%s\n%s" % (r.stdout, r.stderr))
    os.replace(tmp, PEAKS)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
