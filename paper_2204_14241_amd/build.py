"""Build libhmc.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_2204_14241_amd.build   (or build_library() from Python)
"""
import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhmc.so")
SOURCES = [os.path.join(CSRC, f) for f in ("hmc.hip", "fft_f32.hip", "fft_f64.hip", "fft_metric.hip")]
DEPS = SOURCES + sorted(glob.glob(os.path.join(CSRC, "*.h"))) + [
    os.path.join(ROOT, "include", f) for f in ("hmc.h", "hmc_testing.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    # keep packed FP32 instructions out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


def source_hash():
    """First 16 hex digits of the SHA-256 of every source and header the library is built from
    (keys the autotuner's on-disk cache to the kernels it timed)."""
    import hashlib
    h = hashlib.sha256()
    for f in DEPS:
        h.update(os.path.basename(f).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{out}")
    if verbose and out.strip():
        print(out)


def build_library(verbose=False):
    """Compile every HIP source (side by side) and link paper_2204_14241_amd/libhmc.so (always
    rebuilds)."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, os.path.basename(s) + ".o") for s in SOURCES]
        with ThreadPoolExecutor(len(SOURCES)) as pool:
            jobs = [pool.submit(_run, [HIPCC, *FLAGS, f'-DHMC_SOURCE_HASH="{source_hash()}"', "-c", s, "-o", o], verbose)
                    for s, o in zip(SOURCES, objs)]
            for j in jobs:
                j.result()
        _run([HIPCC, f"--offload-arch={ARCH}", "-shared", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    print("built", LIB)
    sys.exit(0)
