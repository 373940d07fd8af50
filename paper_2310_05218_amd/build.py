"""Builds libswconv.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libswconv.so")
BINDING = os.path.join(PKG, "_swnative.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # packed-FP32 VALU forms are switched off for every kernel in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_binding(verbose: bool = False) -> str:
    """Compile the native part of the Python binding (host code against torch's headers) into ``_swnative.so``."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}"]
    for d in [*cpp_extension.include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", d]
    # (torch is imported before the module is: its libraries are found where it loaded them)
    cmd += [os.path.join(CSRC, "binding", "sw_binding.cpp"), "-o", BINDING]
    for d in cpp_extension.library_paths():
        cmd += ["-L", d]
    cmd += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return BINDING


def _build_binding_if_possible(verbose: bool):
    """The binding is optional (without it every call goes through ctypes) and needs torch's headers and a host compiler: where they are
    missing the library is built all the same, and no module of an older build stays beside it."""
    try:
        build_binding(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(BINDING):
            os.remove(BINDING)
        print(f"native binding not built, calls go through ctypes: {e}", file=sys.stderr, flush=True)


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every kernel and the C ABI into ``libswconv.so``; always recompiles.  The translation units
    are compiled side by side into ``_build/`` at the repository root (not tracked), then linked."""
    import concurrent.futures
    import shutil

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    inc = ["-I", os.path.join(PKG, "..", "include")]
    tmp = os.path.join(PKG, "..", "_build")
    shutil.rmtree(tmp, ignore_errors=True)
    os.makedirs(tmp)
    try:
        # the source of the run-time-compiled kernel travels inside the library as a string literal
        with open(os.path.join(CSRC, "jit", "sliding_plane_jit.hip")) as f:
            text = f.read()
        assert ')SWJIT"' not in text
        with open(os.path.join(tmp, "sw_jit_source.inc"), "w") as f:
            f.write('R"SWJIT(' + text + ')SWJIT"\n')
        inc += ["-I", tmp]

        def compile_one(src):
            obj = os.path.join(tmp, os.path.basename(src) + ".o")
            cmd = [hipcc, *HIPCC_FLAGS, *inc, "-c", src, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with concurrent.futures.ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
            binding = pool.submit(_build_binding_if_possible, verbose)
            objs = list(pool.map(compile_one, sources()))
            binding.result()
        cmd = [hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB, *objs, "-lhiprtc"]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
