"""Build libwenoiu.so (HIP, gfx950) in-tree.

hipcc compiles the kernels and the C ABI into paper_1810_11103_amd/libwenoiu.so.
Packed fp32 instructions are disabled for every HIP translation unit.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libwenoiu.so")
SOURCES = ["wiu_kernels.hip", "wiu_stage_kernels.hip", "wiu_batched_kernels.hip", "wiu_adjoint_kernels.hip", "wiu_api.hip",
           "wiu_batched.hip", "wiu_multiblock.hip", "wiu3d.hip"]
HEADERS = ["wiu_device.hpp", "wiu_kernels.hpp", "wiu_sweep.hpp", "wiu_stage.hpp", "wiu_adjoint.hpp", "wiu_mb.hpp"]
ARCH = os.environ.get("WIU_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
]


def _inputs():
    return [os.path.join(CSRC, s) for s in SOURCES + HEADERS] + [os.path.join(INCLUDE, "wenoiu.h")]


def build(force=True, verbose=False):
    """Compile every source; returns the library path."""
    if not force and os.path.exists(LIB) and os.path.getmtime(LIB) >= max(os.path.getmtime(p) for p in _inputs()):
        return LIB
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    for s in SOURCES:
        obj = os.path.join(objdir, s.replace(".hip", ".o"))
        cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, s), "-o", obj]
        if verbose:
            print(" ".join(cmd), file=sys.stderr)
        procs.append(subprocess.Popen(cmd))
        objs.append(obj)
    for p in procs:
        if p.wait() != 0:
            raise RuntimeError("hipcc failed")
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
