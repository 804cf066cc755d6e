"""Build libtaps.so (HIP for gfx950) in-tree.

    python -m paper_2606_00487_amd.build

Every .hip file is compiled to an object with hipcc, the selection kernel with
-ffp-contract=off (its fp64 scores must round every product and sum separately),
the attention kernel with MFMA results in ordinary vector registers; then
everything is linked into paper_2606_00487_amd/libtaps.so.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtaps.so")
ARCH = "gfx950"

COMMON = ["-O3", "-fPIC", "-std=c++17", "-Wall", f"--offload-arch={ARCH}",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
PER_FILE = {
    "select.hip": ["-ffp-contract=off"],
    "api.cpp": ["-ffp-contract=off"],
    # MFMA accumulators in ordinary VGPRs: the attention kernel fits in 256 of them, and
    # the AGPR form would copy its accumulators back and forth around every softmax
    "attn.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
    "attn_f32.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"],
}
SOURCES = ["topk.hip", "select.hip", "attn.hip", "attn_f32.hip", "walk.hip", "commit.hip", "layer.hip",
           "noalloc.hip", "api.cpp"]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    cmd = [hipcc(), *COMMON, *PER_FILE.get(src, []), *lang, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
