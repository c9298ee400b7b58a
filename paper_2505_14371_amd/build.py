"""Compile the HIP sources under csrc/ for gfx950 into libqoda.so next to this file, and the torch-facing loop's native part
(csrc/qoda_torch.cpp, host code only) into _qoda_torch.so where torch, its headers and a host compiler are there."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import warnings

_HERE = os.path.dirname(os.path.abspath(__file__))
SOURCES = [os.path.join(_HERE, "csrc", f) for f in ("qoda_kernels.hip", "qoda_api.hip")]
LIB = os.path.join(_HERE, "libqoda.so")
PROBE_SRC = os.path.join(_HERE, "harness", "qoda_probe.hip")
TORCH_SRC = os.path.join(_HERE, "csrc", "qoda_torch.cpp")
TORCH_LIB = os.path.join(_HERE, "_qoda_torch.so")
PROBE = os.path.join(_HERE, "harness", "qoda_probe")

# -ffp-contract=off: every fp32/fp64 operation that feeds a packed bit stays a single IEEE operation.
# packed-fp32 instructions are switched off for the whole library.
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
               "-fno-fast-math", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall"]


def built_for() -> str:
    """What the native part of the loop is tied to: its code reads the fields of this torch's and this interpreter's objects."""
    import torch

    return f"{torch.__version__} {sysconfig.get_config_var('SOABI')}"


def build_torch(verbose: bool = False) -> str:
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DQODA_BUILT_FOR="{built_for()}"']
    for p in [*include_paths(), sysconfig.get_path("include")]:
        cmd += ["-isystem", p]
    cmd += [TORCH_SRC, "-o", TORCH_LIB] + ["-L" + p for p in library_paths()] + ["-lc10", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    return TORCH_LIB


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *SOURCES, "-o", LIB]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    # the torch-free measurement driver (links the library through its C ABI only)
    cmd = [hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17", PROBE_SRC, "-o", PROBE, "-L" + _HERE, "-lqoda",
           "-Wl,-rpath,$ORIGIN/.."]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    # The library is complete without the rest: where it cannot be built the loop looks at the gradients in Python.
    try:
        build_torch(verbose)
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(TORCH_LIB):
            os.remove(TORCH_LIB)
        warnings.warn(f"{os.path.basename(TORCH_LIB)} was not built ({e}): every gradient is looked at in Python")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
