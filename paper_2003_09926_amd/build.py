"""Build the HIP library libjetles.so in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "_lib")
LIB = os.path.join(LIBDIR, "libjetles.so")
SOURCES = ["jz_stage.hip", "jz_stage32.hip", "jz_brick.hip", "jz_bc.hip", "jz_aux.hip", "jz_api.hip"]
ARCH = os.environ.get("JZ_OFFLOAD_ARCH", "gfx950")

# Packed FP32 instructions are switched off for every device pass.
HIPCC_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wall", "-Wno-unused-result"]


def sources() -> list:
    return [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]


def build_library(verbose: bool = False, extra: list | None = None) -> str:
    """Compile every HIP source into one shared library (always recompiles)."""
    os.makedirs(LIBDIR, exist_ok=True)
    objs, running = [], []
    for src in sources():
        obj = os.path.join(LIBDIR, os.path.basename(src).replace(".hip", ".o"))
        cmd = ["hipcc", *HIPCC_FLAGS, *(extra or []), "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append((cmd, subprocess.Popen(cmd)))   # the sources compile side by side
        objs.append(obj)
    for cmd, proc in running:
        if proc.wait() != 0:
            for _, other in running:
                other.wait()
            raise subprocess.CalledProcessError(proc.returncode, cmd)
    tmp = LIB + ".tmp"
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
