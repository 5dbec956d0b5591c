"""Compile the HIP/C++ sources under csrc/ into liboim.so for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "liboim.so")
OBJ = os.path.join(HERE, "_build")
SOURCES = ["api.cpp", "validate.cpp", "readout.hip", "sparse_persistent.hip",
           "sparse_persistent_uw.hip", "sparse_sorted.hip", "sparse_sorted_uw.hip", "stepwise.hip",
           "dense.hip", "adjoint.hip", "noalloc.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed FP32 VALU forms are disabled for every device compile.
COMMON = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Xclang", "-target-feature",
          "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function",
          "-fvisibility=hidden", "-I", INCLUDE, "-I", CSRC]


# Per-source code generation options: the dense kernel keeps its MFMA
# accumulators in architectural VGPRs (stable allocation, no AGPR copies); the
# host loops of problem creation are aligned, so that their speed does not hang
# on where the linker puts them (30000 oscillators of degree 6 4.85 ms by
# chance, 4.56 ms so; a batch of 256 graphs of 300 10.4 and 9.8 ms).
HOST_ALIGN = ["-falign-functions=64", "-falign-loops=32"]
EXTRA = {"dense.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "api.cpp": HOST_ALIGN, "validate.cpp": HOST_ALIGN}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src + ".o")
    lang = ["-x", "hip"]
    cmd = [HIPCC, *COMMON, *EXTRA.get(src, []), *lang, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
