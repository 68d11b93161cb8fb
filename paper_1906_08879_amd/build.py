"""Builds libplaceto.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libplaceto.so")
SOURCES = ["api.hip", "kernels_generic.hip", "kernels_mfma.hip", "kernels_lanes.hip", "kernels_tiles.hip", "kernels_wide.hip", "kernels_pool_mfma.hip", "kernels_head.hip", "kernels_episode.hip", "kernels_simulator.hip", "kernels_backward.hip", "layout.cpp", "plan.cpp", "workspace.cpp"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # packed fp32 instructions are kept off for every device function
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# Flags of single sources.  Their kernels branch on the scalar unit inside a long dependent chain, and
# structured control flow (which the back end otherwise gives uniform branches too) costs them copies
# of their register state at every join.  (An option of the back end, not of the driver: checked with ROCm 7.2.0,
# clang 22, whose code with and without it gives the same bits on the timed cases.)  Simulator: 3.38 -> 2.70 ms for 256 NASNet-like graphs; sweep:
# forward pass 0.715 -> 0.690 ms (64 NMT-like graphs), 2.16 -> 2.12 ms (256 NASNet-like ones).
_NO_STRUCTURE = ["-mllvm", "-structurizecfg-skip-uniform-regions"]
SOURCE_FLAGS = {"kernels_simulator.hip": _NO_STRUCTURE, "kernels_mfma.hip": _NO_STRUCTURE, "kernels_tiles.hip": _NO_STRUCTURE, "kernels_wide.hip": _NO_STRUCTURE, "kernels_lanes.hip": _NO_STRUCTURE}


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compiles every source to an object (in parallel) and links libplaceto.so."""
    from concurrent.futures import ThreadPoolExecutor
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    common = [hipcc(), *flags, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC]

    def compile_one(src: str) -> str:
        obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
        cmd = common + ["-c"] + (["-x", "hip"] if src.endswith(".cpp") else []) + SOURCE_FLAGS.get(src, []) + [os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES), os.cpu_count() or 1)) as pool:
        objs = list(pool.map(compile_one, SOURCES))
    cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra_flags=sys.argv[1:]))
