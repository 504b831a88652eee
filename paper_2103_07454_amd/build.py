"""Compiles the HIP sources under ``csrc/`` into ``libevg.so`` for gfx950."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libevg.so")
SOURCES = ["evg_api.hip", "kernels_update.hip", "kernels_walk.hip", "kernels_parts.hip", "kernels_ring.hip", "kernels_trigger.hip", "kernels_topk.hip", "kernels_choose.hip"]

# -ffp-contract=off: every fused multiply-add in the kernels is written out, so
#   results do not depend on what the compiler decides to contract.
# correctly rounded divide/sqrt: the generator relies on IEEE results.
# packed fp32 ops are switched off (scalar fp32 code only).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"] + os.environ.get("EVG_EXTRA_FLAGS", "").split()


def build_library(verbose: bool = False) -> str:
    objs = []

    def compile_one(src):
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
