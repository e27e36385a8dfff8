"""Build libgrinqh.so in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgrinqh.so")
SOURCES = ["grinqh_api.hip", "pack.hip", "assign.hip", "vmm.hip", "vmm_dot2.hip", "vmm_pp.hip",
           "vmm_mm.hip", "prefill.hip", "prefill_small.hip", "vmm_lut.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-fvisibility=hidden", "-Wall", "-Wno-unused-result", "-Werror=inline-asm",
    # keep the compiler from forming packed fp32 arithmetic on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


# per-source extra flags: prefill.hip and vmm_mm.hip keep their fixed-size register
# arrays in registers (the compiler would otherwise place some in LDS, which
# their tiles need); vmm_pp.hip and vmm_mm.hip preload their first kernel arguments
SOURCE_FLAGS = {"prefill.hip": ["-mllvm", "-disable-promote-alloca-to-lds"],
                # the batch-1 kernels' leading arguments (x, level map, groups)
                # arrive in scalar registers at wave launch, so the first load
                # of x does not wait for a kernel-argument load
                "vmm_mm.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=16",
                               "-mllvm", "-disable-promote-alloca-to-lds"],
                "vmm_pp.hip": ["-mllvm", "-amdgpu-kernarg-preload-count=16"]}


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source and link libgrinqh.so; returns the library path."""
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    for src in SOURCES:
        obj = os.path.join(BUILD, src.replace(".hip", ".o"))
        cmd = [hipcc(), *HIPCC_FLAGS, *SOURCE_FLAGS.get(src, []), *extra_flags, "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError(f"hipcc failed on {src}")
        # warnings; the host pass does not know the packed-fp32 feature, which is harmless
        sys.stderr.writelines(l for l in r.stderr.splitlines(True) if "'-packed-fp32-ops' is not a recog" not in l)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libgrinqh.so failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
