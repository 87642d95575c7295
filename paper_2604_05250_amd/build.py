"""Build the HIP library (libdd.so, hipcc for gfx950) and the native part of the Python binding (_binding.so, g++) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libdd.so")
SOURCES = ["dd_api.hip", "verify.hip", "attention_mfma.hip", "attention_wide.hip", "attention_stream.hip", "attention_duo.hip", "attention_solo.hip", "attention_f32.hip", "cache.hip"]
HEADERS = ["dd_internal.h", "attention_common.h", os.path.join("..", "..", "include", "dd.h")]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-Wall", "-Wno-unused-function", "-Wno-inline-asm",
         # packed-fp32 instructions are kept out of the generated code: some of their forms have given wrong results
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # leading scalar kernel arguments (up to fourteen words) are in registers when a wave starts, not fetched by it
         "-mllvm", "-amdgpu-kernarg-preload-count=16"]


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in SOURCES + HEADERS]
    return any(os.path.getmtime(p) > t for p in deps)


def build_library(force: bool = True, verbose: bool = False, extra_flags=()) -> str:
    """Compile every kernel source into one shared library.  Returns its path."""
    if not force and not stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + FLAGS + list(extra_flags) + ["-o", LIB] + [os.path.join(CSRC, f) for f in SOURCES]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return LIB


BINDING = os.path.join(_HERE, "_binding.so")
BINDING_SOURCE = os.path.join(CSRC, "binding.cpp")


def build_binding(verbose: bool = False) -> str:
    """Compile the binding's native part against torch's headers; it loads libdd.so from its own directory."""
    import sysconfig

    import torch
    t = os.path.dirname(os.path.abspath(torch.__file__))
    inc = [os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
           os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include"), sysconfig.get_paths()["include"]]
    lib = os.path.join(t, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    cmd += [x for d in inc for x in ("-isystem", d)] + ["-o", BINDING, BINDING_SOURCE, "-L" + _HERE, "-l:" + os.path.basename(LIB)]
    cmd += ["-L" + lib, "-lc10", "-lc10_hip", "-ltorch_hip", "-ltorch_cpu", "-ltorch_python", "-lamdhip64", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stdout)
    if verbose and res.stdout.strip():
        print(res.stdout)
    return BINDING


if __name__ == "__main__":
    print(build_library(force=True, verbose=True, extra_flags=sys.argv[1:]))
    print(build_binding(verbose=True))
