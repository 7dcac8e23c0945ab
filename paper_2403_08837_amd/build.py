"""Builds libcdp.so (HIP kernels + host engine + C ABI) in-tree for gfx950, and _calls.so, its kernel-level entry points as Python calls."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcdp.so")
CALLS = os.path.join(HERE, "_calls.so")
SOURCES = ["gemm.hip", "linear_kernels.hip", "gemm_stream.hip", "conv_kernels.hip", "conv256_kernels.hip", "conv_wgrad_small.hip", "small_kernels.hip", "transformer_kernels.hip", "attention_kernels.hip", "static_scratch.hip", "engine.cpp", "host_copy.cpp", "plan.cpp", "kernels_api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 VALU forms are switched off for all device code: the compiler then emits scalar fp32 ops only
# fp32 atomic adds go to coarse-grained device memory (the arena): use the hardware instruction, not a CAS loop
DEVICE_FLAGS = ["--offload-arch=gfx950", "-munsafe-fp-atomics", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-D__HIP_PLATFORM_AMD__"]


def build(verbose: bool = False) -> str:
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src + ".o")
        cmd = [HIPCC] + COMMON + (DEVICE_FLAGS if src.endswith(".hip") else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        # hipcc compiles every .hip file twice; the HOST (x86-64) pass does not know the AMDGPU feature name and says
        # "'-packed-fp32-ops' is not a recognized feature for this target (ignoring feature)".  The device pass takes it.
        out = "\n".join(l for l in out.splitlines() if "is not a recognized feature for this target" not in l)
        if p.returncode != 0:
            failed = True
            print("---- %s failed ----\n%s" % (src, out), file=sys.stderr)
        elif out.strip() and verbose:
            print(out)
    if failed:
        raise RuntimeError("libcdp build failed")
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    build_calls(verbose)
    return LIB


def build_calls(verbose: bool = False) -> None:
    """_calls.so saves a kernel-level call one to two microseconds; without a C++ compiler or Python's headers those calls go through
    ctypes."""
    if os.path.exists(CALLS):
        os.remove(CALLS)  # not one of another build
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-shared", "-I" + sysconfig.get_paths()["include"],
           os.path.join(CSRC, "pycalls.cpp"), "-o", CALLS]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        subprocess.run(cmd, check=True)
    except (OSError, subprocess.CalledProcessError) as e:
        print("_calls.so was not built (%s): kernel-level calls go through ctypes" % e, file=sys.stderr)


if __name__ == "__main__":
    print(build(verbose=True))
