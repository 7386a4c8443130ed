"""Build the gfx950 shared library (libtensorbleu.so) and the Python module that calls it in-tree.

`python -m paper_2510_05485_amd.build` compiles every HIP translation unit under csrc/ for
gfx950 and links them into one C-ABI library next to this file, and csrc/tb_host.cpp (host code,
against PyTorch's headers) into the module _host.  hipcc cross-compiles without a GPU, so this runs
anywhere the ROCm toolchain is installed.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libtensorbleu.so")
HOST_SRC = os.path.join(CSRC, "tb_host.cpp")
HOST_LIB = os.path.join(PKG, "_host.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PRELOADED_WORDS = 14  # of a kernel's plain arguments
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first 56 bytes of a kernel's plain arguments come in scalar registers
    "-mllvm", f"-amdgpu-kernarg-preload-count={PRELOADED_WORDS}", f"-DTB_PRELOADED_WORDS={PRELOADED_WORDS}",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(HOST_LIB):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(HOST_LIB))
    deps = sources() + [HOST_SRC] + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build(verbose: bool = True) -> str:
    tmp = LIB + f".tmp{os.getpid()}"
    extra = os.environ.get("TB_HIPCC_EXTRA", "").split()   # extra hipcc flags for experiments
    include = ["-I", INCLUDE, "-I", CSRC]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    # (the files side by side: 100 s instead of 180, of which tb_fused.hip takes nearly all)
    with tempfile.TemporaryDirectory() as objects, concurrent.futures.ThreadPoolExecutor(4) as pool:
        names = [os.path.join(objects, os.path.basename(f) + ".o") for f in sources()]
        list(pool.map(run, [[HIPCC, *FLAGS, *extra, *include, "-c", f, "-o", o] for f, o in zip(sources(), names)]))
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", "-o", tmp, *names])
    os.replace(tmp, LIB)
    build_host(verbose)
    return LIB


def build_host(verbose: bool = True) -> str:
    """The module _host: links against the library and PyTorch."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    include = [INCLUDE, *cpp_extension.include_paths(), os.path.join(rocm, "include"),
               sysconfig.get_paths()["include"]]
    tmp = HOST_LIB + f".tmp{os.getpid()}"
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-isystem{d}" for d in include], "-o", tmp, HOST_SRC, "-L", PKG, "-ltensorbleu",
           "-L", torch_lib, "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
           "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, HOST_LIB)
    return HOST_LIB


EXAMPLE_SRC = os.path.join(PKG, "example", "c_caller.c")
EXAMPLE_BIN = os.path.join(PKG, "c_caller")


def build_example(verbose: bool = True) -> str:
    """The plain-C caller of the ABI (gcc, HIP runtime only), linked against the library."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = [os.environ.get("CC", "gcc"), "-std=c99", "-O2", "-Wall", "-D__HIP_PLATFORM_AMD__",
           "-I", INCLUDE, "-I", os.path.join(rocm, "include"), EXAMPLE_SRC, "-L", PKG,
           "-ltensorbleu", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-lm",
           "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", EXAMPLE_BIN]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return EXAMPLE_BIN


if __name__ == "__main__":
    build()
    build_example()
    print("built", LIB)
    sys.exit(0)
