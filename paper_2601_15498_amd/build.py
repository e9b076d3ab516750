"""Compile the HIP library (csrc/mars.hip) for gfx950 into paper_2601_15498_amd/libmars.so, and the native part of its
Python binding (csrc/marshal.cpp) into paper_2601_15498_amd/_marshal.so."""
import os
import subprocess
import sys
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "mars.hip")
LIB = os.path.join(HERE, "libmars.so")
MARSHAL_SRC = os.path.join(HERE, "csrc", "marshal.cpp")
MARSHAL_LIB = os.path.join(HERE, "_marshal.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-shared", "-fPIC",
    # compiler-generated packed fp32 arithmetic is switched off for every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # device code never sees NaN (a stated precondition): without this every fmax/med3 operand
    # is first canonicalised by an extra v_max, doubling the per-element work of the row reduction
    "-Xarch_device", "-fno-honor-nans",
    "-Wall", "-Wno-unused-function",
]


def build_marshal(verbose: bool = False, out: str = MARSHAL_LIB, extra=()) -> str:
    import sysconfig
    import torch
    from torch.utils.cpp_extension import include_paths
    include = [sysconfig.get_paths()["include"]] + [p for p in include_paths() if os.path.isdir(p)]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DMARS_TORCH_VERSION="{torch.__version__}"']
    cmd += ["-isystem" + p for p in include] + list(extra) + ["-o", out, MARSHAL_SRC]
    cmd += ["-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out


def build(verbose: bool = False, extra=()) -> str:
    cmd = [HIPCC] + FLAGS + list(extra) + ["-o", LIB, SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    # The binding does without its native part where this machine cannot build it (no g++, no Python.h).
    if os.path.exists(MARSHAL_LIB):
        os.remove(MARSHAL_LIB)
    try:
        build_marshal(verbose)
    except (OSError, subprocess.CalledProcessError) as e:
        warnings.warn(f"{MARSHAL_LIB} was not built ({e}): calls will go through ctypes", RuntimeWarning)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
