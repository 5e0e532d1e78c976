"""Compile the HIP library (Go and Hex kernels) for gfx950 into paper_2303_17503_amd/libpgxgo.so and the host extension _fastcall.so (in-tree)."""
import os
import subprocess
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRCS = [os.path.join(HERE, "csrc", "pgxgo.hip"), os.path.join(HERE, "csrc", "pgxhex.hip")]
LIB = os.path.join(HERE, "libpgxgo.so")
FAST = os.path.join(HERE, "_fastcall.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def build(verbose: bool = False) -> str:
    cmd = [
        HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-mllvm", "-amdgpu-kernarg-preload-count=16",   # leading kernel arguments in scalar registers (wave_common.hpp)
        "-Wall", "-Wno-unused-command-line-argument",
        "-I", os.path.join(ROOT, "include"), "-o", LIB, *SRCS,
    ]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout)
    if verbose and out.strip():
        print(out)
    try:
        build_fastcall(verbose)
    except (RuntimeError, OSError, ImportError) as e:   # the library is whole without it: binding.py then checks in Python
        warnings.warn(f"{os.path.basename(FAST)} was not built: {e}", RuntimeWarning)
    return LIB


def build_fastcall(verbose: bool = False) -> str:
    """The native argument checks of the per-ply calls (a CPython extension against this torch)."""
    if os.path.exists(FAST):   # never an older one beside a newer library
        os.remove(FAST)
    import torch
    from torch.utils import cpp_extension

    libs = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [
        "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
        *[f"-I{p}" for p in cpp_extension.include_paths()], "-I" + sysconfig.get_paths()["include"],
        "-o", FAST, os.path.join(HERE, "csrc", "fastcall.cpp"), f"-L{libs}", "-lc10", "-ltorch_cpu", "-ltorch_python", f"-Wl,-rpath,{libs}",
    ]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed:\n" + r.stdout)
    return FAST


if __name__ == "__main__":
    print(build(verbose=True))
