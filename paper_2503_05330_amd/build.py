"""Compiles the HIP sources under csrc/ into libcsd.so (gfx950 only)."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))
LIBRARY = os.path.join(HERE, "libcsd.so")

# -packed-fp32-ops is switched off on purpose: the compiler must not form packed
# FP32 instructions from ordinary float code in this library.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build_library() -> str:
    """One object per source, compiled side by side, and one link."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        raise RuntimeError("hipcc not found: the csd HIP library cannot be built")
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]

        def compile_one(pair):
            source, obj = pair
            subprocess.check_call([hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"),
                                   "-c", "-o", obj, source])

        with ThreadPoolExecutor(max_workers=min(16, os.cpu_count() or 1)) as pool:
            list(pool.map(compile_one, zip(SOURCES, objects)))
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIBRARY, *objects])
    return LIBRARY


if __name__ == "__main__":
    print(build_library())
