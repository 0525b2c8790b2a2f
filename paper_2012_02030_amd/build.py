"""Build the gfx950 shared library (hipcc cross-compiles without a GPU) and the binding's native call path."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libap_mi355x.so")
CALLS = os.path.join(PKG, "ap_calls.so")                      # torch tensors -> C-ABI call (host code)
RESOURCES = os.path.join(PKG, "libap_mi355x.resources.txt")   # per-kernel registers, spills, LDS

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # leading scalar kernel arguments (up to 16 dwords) arrive in registers when a wavefront starts
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
    # a constant that does not fit the type it is converted to is an error, not a value
    "-Werror=literal-conversion",
    # the LDS-direct load helper names M0 as clobbered; the compiler remarks that M0 is a reserved
    # register (it never keeps a value of its own live in it across a statement)
    "-Wno-inline-asm",
    "-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def kernel_resources(compiler_output: str) -> list:
    """Per-kernel figures from the compiler's resource-usage remarks: one dict per kernel."""
    kernels, cur = [], None
    for line in compiler_output.splitlines():
        if "remark:" not in line:
            continue
        text = line.split("remark:", 1)[1].split("[-Rpass", 1)[0].strip()
        if text.startswith("Function Name:"):
            cur = {"name": text.split(":", 1)[1].strip()}
            kernels.append(cur)
        elif cur is not None and ":" in text:
            key, val = text.split(":", 1)
            cur[key.strip()] = val.strip()
    return kernels


def build(verbose: bool = False, extra=()) -> str:
    """Compile every HIP source into libap_mi355x.so next to this file and return its path.

    Writes the per-kernel register, spill and LDS figures next to the library and warns if any
    kernel spills vector registers: spilled values travel through the same in-order vector memory
    path as the tile loads, and a reload inside a tile loop then waits for the tiles in flight
    (tests/test_abi.py asserts that there is none)."""
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [HIPCC, *FLAGS, *extra, *sources(), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only target feature and says so; drop that line
    out = "\n".join(line for line in proc.stdout.splitlines() if "packed-fp32-ops" not in line)
    if proc.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("hipcc failed:\n" + out)
    kernels = kernel_resources(out)
    out = "\n".join(line for line in out.splitlines() if "-Rpass-analysis=kernel-resource-usage" not in line)
    if verbose and out.strip():
        print(out)
    with open(RESOURCES, "w") as f:
        for k in kernels:
            f.write("%s  VGPRs %s  AGPRs %s  spilled VGPRs %s  spilled SGPRs %s  waves/SIMD %s  LDS %s\n" % (
                k["name"], k.get("VGPRs", "?"), k.get("AGPRs", "?"), k.get("VGPRs Spill", "?"),
                k.get("SGPRs Spill", "?"), k.get("Occupancy [waves/SIMD]", "?"),
                k.get("LDS Size [bytes/block]", "?")))
    spilling = [k["name"] for k in kernels if k.get("VGPRs Spill", "0") != "0"]
    if spilling:                                             # the library still works; the tests flag it
        print("WARNING: kernels that spill vector registers: " + ", ".join(spilling), flush=True)
    os.replace(tmp, LIB)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False):
    """Compile the CPython module that takes the attention calls from torch tensors to the library.

    It saves host time and nothing else needs it, so where there is no host compiler or no headers the library stands
    without it (and without an old one, which may be of another C ABI); returns None then."""
    import torch
    tdir = os.path.dirname(os.path.abspath(torch.__file__))
    cxx = os.environ.get("CXX", "g++")
    needs = [os.path.join(sysconfig.get_paths()["include"], "Python.h"),
             os.path.join(tdir, "include", "torch", "csrc", "autograd", "python_variable.h")]
    missing = [n for n in needs if not os.path.exists(n)] + ([] if shutil.which(cxx) else [cxx])
    if missing:
        print("WARNING: the native call path is not built, missing: " + ", ".join(missing), flush=True)
        if os.path.exists(CALLS):
            os.remove(CALLS)
        return None
    tmp = CALLS + ".tmp.%d" % os.getpid()
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I", os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"],
           "-isystem", os.path.join(tdir, "include"),
           "-isystem", os.path.join(tdir, "include", "torch", "csrc", "api", "include"),
           os.path.join(CSRC, "ap_calls.cpp"), "-L", os.path.join(tdir, "lib"),
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("building the call path failed:\n" + proc.stdout)
    os.replace(tmp, CALLS)
    return CALLS


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
