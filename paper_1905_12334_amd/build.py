"""Build, in-tree, libmp8.so (the HIP library behind the C ABI in include/mp8.h, for gfx950) and the
extension module _binding (host code only: torch tensors to calls of that ABI)."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmp8.so")
SOURCES = ["quantize.hip", "update.hip", "gemm.hip", "host.hip"]
# -ffp-contract=off: every multiply and add is rounded on its own (the one fused operation,
# the weight update, is an explicit fma).  Packed FP32 instructions are switched off.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall",
         "-Wno-unused-command-line-argument",
         # the direct-to-LDS load names M0 as clobbered; clang remarks that M0 is a reserved register
         "-Wno-inline-asm",
         # "#pragma unroll(expression)" with a template-dependent count is meant as written
         "-Wno-cuda-compat"]


def build_binding(verbose: bool = False) -> str:
    """The extension module: plain C++ against torch's and Python's headers.  It is linked against
    torch's libraries by name only; the package imports torch, and with it these libraries, first."""
    import torch
    from torch.utils import cpp_extension
    lib = os.path.join(HERE, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))
    inc = [*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"]]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *(f"-isystem{i}" for i in inc),
           os.path.join(CSRC, "binding.cpp"), "-o", lib, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return lib


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        objs.append(obj)
    build_binding(verbose)
    for cmd, p in procs:
        out, _ = p.communicate()
        text = "\n".join(l for l in out.decode().splitlines()
                         if "is not a recognized feature" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + text)
        if verbose and text.strip():
            print(text)
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(link, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
