"""Build libralm.so (hand-written HIP for gfx950) in-tree with hipcc.

Usage: ``python -m paper_2401_14021_amd.build``.  Each translation unit is compiled on
its own (in parallel) and linked into ``paper_2401_14021_amd/libralm.so``.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libralm.so")
SOURCES = ["ralm_api.hip", "scan_kernels.hip", "scan_held_kernels.hip", "select_kernels.hip", "cache_verify_kernels.hip", "knnlm_kernels.hip",
           "os3_host.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the scan kernel's stage bodies are fully unrolled by design (static register indices)
         "-mllvm", "-pragma-unroll-threshold=1000000"]


# Matrix results in vector registers: the kernel fills the accumulation registers with its queries.  An option of the compiler's
# back end (ROCm 7.2); one that does not know it refuses this file.
EXTRA = {"scan_held_kernels.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build() -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build())
