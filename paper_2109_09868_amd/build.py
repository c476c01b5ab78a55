"""Compile the HIP sources into paper_2109_09868_amd/libapproxifer.so for gfx950, and the binding's marshalling module."""
from __future__ import annotations

import os
import shutil
import subprocess

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libapproxifer.so")
SOURCES = ["api.hip", "encode.hip", "decode.hip", "byzantine.hip", "byzantine_pairs_large.hip",
           "byzantine_null_pairs_large.hip", "byzantine_pairs_medium.hip", "byzantine_null_pairs_medium.hip",
           "byzantine_pairs_small.hip", "byzantine_null_pairs_small.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc_path() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the library cannot be built")
    return exe


def host_compiler() -> str:
    """g++, or where there is none the compiler that hipcc itself drives."""
    exe = shutil.which("g++")
    if exe is None:
        rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path())))
        exe = os.path.join(rocm, "llvm", "bin", "clang++")
    return exe


def build_marshal(verbose: bool = False, out: str = os.path.join(PKG_DIR, "_marshal.so")) -> str:
    """Compile csrc/marshal.cpp (host code on torch's C++ interface) into the module paper_2109_09868_amd._marshal."""
    import sysconfig

    import torch
    from torch.utils import cpp_extension

    from . import binding

    include = [os.path.join(ROOT, "include"), *cpp_extension.include_paths(), sysconfig.get_paths()["include"],
               os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path()))), "include")]
    cmd = [host_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DAPPROXIFER_BUILT_FOR="%s"' % binding.marshal_target(), *("-I" + p for p in include),
           os.path.join(CSRC, "marshal.cpp"), "-o", out, *("-L" + p for p in cpp_extension.library_paths()),
           "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed on marshal.cpp:\n%s\n%s" % (cmd[0], r.stdout, r.stderr))
    return out


def build_library(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source (in parallel, one hipcc per file) and link the shared library."""
    from concurrent.futures import ThreadPoolExecutor

    hipcc = hipcc_path()
    objdir = os.path.join(PKG_DIR, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, *inc, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
    print(build_marshal(verbose=True))
