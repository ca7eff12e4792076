"""Builds the HIP library in-tree: paper_2601_20499_amd/libdf_hip.so (gfx950 only), and where the machine has what it takes the
extension that marshals the binding's frequent calls."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libdf_hip.so")
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))   # for this interpreter alone
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


def marshal_includes(torch_dir: str):
    return [os.path.join(torch_dir, "include"), sysconfig.get_paths()["include"], "/opt/rocm/include"]


def marshal_lacks() -> list:
    """What this machine lacks of what the extension is built with."""
    lacks = [] if shutil.which("g++") else ["g++"]
    try:
        import torch
    except ImportError:
        return lacks + ["torch"]
    headers = ("torch/csrc/autograd/python_variable.h", "c10/hip/HIPStream.h", "Python.h", "hip/hip_runtime_api.h")
    include = marshal_includes(os.path.dirname(torch.__file__))
    return lacks + [h for h in headers if not any(os.path.exists(os.path.join(i, h)) for i in include)]


def marshal_command(out: str = MARSHAL):
    """The Python extension of the binding (host code only; it takes torch tensors)."""
    import torch
    t = os.path.dirname(torch.__file__)
    include = [*marshal_includes(t), os.path.join(ROOT, "include")]
    return (["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [x for i in include for x in ("-isystem", i)] +
            [os.path.join(CSRC, "df_marshal.cpp"), "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
             "-Wl,-rpath," + os.path.join(t, "lib"), "-o", out])


def build_library(verbose: bool = True, extra=()) -> str:
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True, cwd=CSRC)

    run(hipcc_command(extra=extra))
    # one of an earlier build may not go with this library; without any the binding marshals its calls in Python
    for old in (MARSHAL, os.path.join(PKG, "_marshal.so")):
        if os.path.exists(old):
            os.remove(old)
    lacks = marshal_lacks()
    if lacks:
        print("the binding's extension is not built, calls are marshalled in Python: no " + ", ".join(lacks), flush=True)
    else:
        run(marshal_command(MARSHAL))
    return LIB


if __name__ == "__main__":
    build_library(extra=sys.argv[1:])
