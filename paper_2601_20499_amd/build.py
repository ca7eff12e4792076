"""Builds the HIP library in-tree: paper_2601_20499_amd/libdf_hip.so (gfx950 only)."""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libdf_hip.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
SOURCES = ["df_host.cpp", "df_cache.hip", "df_attn.hip"]


def hipcc_command(out: str = LIB, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
           # packed fp32 VALU forms are kept out of the generated code on purpose
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    cmd += list(extra)
    for s in SOURCES:
        path = os.path.join(CSRC, s)
        cmd += (["-x", "hip", path] if s.endswith(".hip") else ["-x", "c++", path])
    cmd += ["-o", out]
    return cmd


def marshal_command(out: str = MARSHAL):
    """The Python extension of the binding (host code only; it takes torch tensors)."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    include = [os.path.join(t, "include"), sysconfig.get_paths()["include"], "/opt/rocm/include", os.path.join(ROOT, "include")]
    return (["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [x for i in include for x in ("-isystem", i)] +
            [os.path.join(CSRC, "df_marshal.cpp"), "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
             "-Wl,-rpath," + os.path.join(t, "lib"), "-o", out])


def build_library(verbose: bool = True, extra=()) -> str:
    for cmd in (hipcc_command(extra=extra), marshal_command()):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, cwd=CSRC)
    return LIB


if __name__ == "__main__":
    build_library(extra=sys.argv[1:])
