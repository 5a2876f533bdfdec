"""Compiles the HIP sources under csrc/ into libcsd.so (gfx950 only), and the native part of the
PyTorch binding."""
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
BINDING = os.path.join(HERE, "_csd_torch.so")

# -packed-fp32-ops is switched off on purpose: the compiler must not form packed
# FP32 instructions from ordinary float code in this library.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build_library() -> str:
    """One object per source, compiled side by side, and one link; then the binding on top of it."""
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
    build_binding()
    return LIBRARY


def timing_source() -> str:
    """All sources as one, for the timing build: its kernels write their clock stamps to a device
    array of the source that they are in, and csd_read_stamps reads that of csd.hip."""
    return "#define CSD_STAMPS 1\n" + "".join(
        '#define launch launch_%d\n#include "%s"\n#undef launch\n' % pair for pair in enumerate(SOURCES))


def build_timing_library(path: str, flags=("-shared",)) -> str:
    """The library with the clock stamps in its kernels (a quarter of an hour: one source)."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    with tempfile.TemporaryDirectory() as tmp:
        source = os.path.join(tmp, "timing.hip")
        with open(source, "w") as f:
            f.write(timing_source())
        subprocess.check_call([hipcc, *HIPCC_FLAGS, "-I", os.path.join(ROOT, "include"), *flags, "-o", path, source])
    return path


def build_binding() -> str:
    """_csd_torch.so, linked to libcsd.so beside it."""
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    gxx = shutil.which("g++") or "/usr/bin/g++"
    includes = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], *include_paths()]
    libs = library_paths()
    subprocess.check_call([gxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
                           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                           *[x for i in includes for x in ("-isystem" if i != includes[0] else "-I", i)],
                           os.path.join(HERE, "csrc", "binding.cpp"), "-o", BINDING,
                           *["-L" + p for p in libs], "-L" + HERE, "-l:libcsd.so", "-lc10", "-ltorch_cpu", "-ltorch",
                           "-ltorch_python", "-Wl,-rpath,$ORIGIN"])
    return BINDING


if __name__ == "__main__":
    print(build_library())
