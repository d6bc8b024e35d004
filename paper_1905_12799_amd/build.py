"""Builds librls.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librls.so")
SOURCES = ["rls_api.hip", "gbt_score.hip", "kmeans_seed.hip", "kmeans_order.hip", "kmeans_lloyd.hip", "kmeans_small.hip", "snap.hip", "modes_visited.hip",
           "sweep_static.hip", "matrix_step.hip"]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, "rls_internal.h"), os.path.join(CSRC, "lloyd_device.h"), os.path.join(ROOT, "include", "rls.h"),
                        os.path.join(ROOT, "include", "rls_bench.h")]
    return any(os.path.getmtime(p) > t for p in deps)


def build_library(verbose: bool = False) -> str:
    """Compile every kernel file for gfx950, side by side, and link the shared library. Always compiles."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off", "-mllvm", "-amdgpu-mfma-vgpr-form",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC]
    # the Lloyd kernels of the larger padded numbers of features are objects of their own (they take longest and go first)
    lloyd = os.path.join(CSRC, "kmeans_lloyd.hip")
    units = [(lloyd, ["-DRLS_LLOYD_DPAD=32"]), (lloyd, ["-DRLS_LLOYD_DPAD=16"]), (lloyd, [])] + [(s, []) for s in sources() if s != lloyd]
    noise = "is not a recognized feature for this target"

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(line for line in res.stderr.splitlines() if noise not in line)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, f"{i}.o") for i in range(len(units))]
        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(lambda unit, obj: run([hipcc] + flags + unit[1] + ["-c", "-o", obj, unit[0]]), units, objects))
        run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", "-o", LIB] + objects)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
