"""Builds libpackkv.so (HIP, gfx950 only) in-tree with hipcc, and the binding's native part with g++.  The library works
without that part, whose name says which Python and torch it was built against."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpackkv.so")
NATIVE_SOURCE = os.path.join(CSRC, "binding_native.cpp")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-ffp-contract=off",                          # FMAs only where written
    "-fhip-fp32-correctly-rounded-divide-sqrt",   # quantizer needs IEEE divide
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form",           # MFMA accumulators stay in VGPRs (no AGPR copies)
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def native_path() -> str:
    """The module that marshals the binding's frequent calls, as built against this Python and this torch."""
    import torch
    return os.path.join(HERE, "_native-%s-torch%s.so" % (sys.implementation.cache_tag, torch.__version__))


def build_native(verbose: bool = False) -> str:
    """Compile that module (against torch's headers)."""
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    native = native_path()
    tmp = native + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-isystem", os.path.join(base, "include"), "-I", sysconfig.get_paths()["include"], "-o", tmp, NATIVE_SOURCE,
           "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    os.replace(tmp, native)
    return native


def build(verbose: bool = False) -> str:
    """Compile every HIP source (one hipcc process per file, in parallel) and link them into one
    shared library, and the native module beside it (without a compiler or headers for that one the binding works in
    Python alone); always recompiles."""
    import concurrent.futures
    import shutil
    import tempfile
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-shared"] + os.environ.get("PACKKV_EXTRA_FLAGS", "").split()
    flags += ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objdir = tempfile.mkdtemp(prefix="packkv_build_")
    try:
        def compile_one(src):
            obj = os.path.join(objdir, os.path.basename(src) + ".o")
            cmd = [hipcc] + flags + ["-c", "-o", obj, src]
            if verbose:
                print(" ".join(cmd))
            subprocess.check_call(cmd)
            return obj
        jobs = max(1, min(len(sources()), int(os.environ.get("MAX_JOBS", "0")) or os.cpu_count() or 1, 8))
        with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
            native = pool.submit(build_native, verbose)
            objs = list(pool.map(compile_one, sources()))
            try:
                native.result()
            except (OSError, subprocess.CalledProcessError) as e:
                warnings.warn("the binding's native part was not built: %s" % e)
        tmp = LIB + ".tmp%d" % os.getpid()
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
        if verbose:
            print(" ".join(cmd))
        subprocess.check_call(cmd)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(objdir, ignore_errors=True)
    return LIB


def stale() -> bool:
    native = native_path()
    if not (os.path.exists(LIB) and os.path.exists(native)):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(native))
    deps = sources() + [NATIVE_SOURCE] + glob.glob(os.path.join(CSRC, "*.h")) + [os.path.join(ROOT, "include", "packkv.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build(verbose=True))
