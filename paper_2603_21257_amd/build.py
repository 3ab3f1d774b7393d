"""Builds libcalvo.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libcalvo.so")
SOURCES = ["calvo_api.hip", "calvo_dispatch.hip", "kernels_ingest.hip", "attn_rows.hip", "attn_pipe.hip", "attn_duo.hip", "mfma_peak.hip", "attn_plan.cpp", "ingest_plan.cpp", "calvo_sched.cpp", "calvo_pool.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # MFMA results in architectural registers unless the allocator finds no room there: in accumulation registers, the
         # compiler's choice for the widest packed-rows kernels (attn_rows.hip), every score and sum that vector instructions
         # touch is moved over and back.  8192+512 tokens, 32Q/8KV: fp32 D = 128 656 -> 608 us, D = 256 1647 -> 1570, bf16
         # D = 256 649 -> 634; the kernels below 256 registers come out the same.
         "-mllvm", "-amdgpu-mfma-vgpr-form",
         "-Wno-unused-result", "-fno-gpu-rdc"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 feature; that is harmless
    out = "\n".join(ln for ln in res.stdout.splitlines() if "packed-fp32-ops" not in ln)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
