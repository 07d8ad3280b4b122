"""Builds libhlbm.so (gfx950 HIP kernels + C ABI) in-tree with hipcc, and
libhlbm_canary.so, the same sources with 64 x 4 tiles and every sweep's
workgroup order flipped (XCD-renumbered where the default keeps the dispatch
order and the other way round): the race canary, under which every per-cell
result must be bitwise the same.  It also takes multi-step passes on every
lattice that can, whether they pay there or not."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libhlbm.so")
CANARY_PATH = os.path.join(HERE, "libhlbm_canary.so")
SOURCES = ["hlbm_launch.hip", "hlbm_march2d.hip", "hlbm_march2d_adjoint.hip", "hlbm_march3d.hip", "hlbm_march3d_adjoint.hip",
           "hlbm_window2d.hip", "hlbm_packed2d.hip", "hlbm_api.hip"]
ARCH = os.environ.get("HLBM_OFFLOAD_ARCH", "gfx950")
CANARY_DEFINES = ["-DHLBM_TILE_BX=64", "-DHLBM_XCD_REMAP=0", "-DHLBM_PASS_RULES=0"]


FLAGS = [
    "-O3", f"--offload-arch={ARCH}", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # multiply-adds fused per source expression only, so the same inlined
    # per-cell code rounds identically in every kernel that contains it
    "-ffp-contract=on",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build(verbose: bool = False, canary: bool = True) -> str:
    """Compiles every source of both libraries (one object each, in parallel),
    then links them."""
    libs = [(LIB_PATH, [])] + ([(CANARY_PATH, CANARY_DEFINES)] if canary else [])
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
            # the host pass warns about the device-only target feature; keep other diagnostics
            err = "\n".join(l for l in p.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
            if err and (verbose or p.returncode != 0):
                sys.stderr.write(err + "\n")
            return p.returncode == 0

        jobs = []
        for i, (out, defines) in enumerate(libs):
            for s in SOURCES:
                obj = os.path.join(tmp, f"{i}_{s}.o")
                jobs.append((out, obj, pool.submit(run, ["hipcc", *FLAGS, *defines, "-c", "-o", obj,
                                                         os.path.join(CSRC, s)])))
        if not all([j.result() for _, _, j in jobs]):
            raise RuntimeError("hipcc failed building the HLBM library")
        for out, _ in libs:
            objs = [o for lib, o, _ in jobs if lib == out]
            if not run(["hipcc", f"--offload-arch={ARCH}", "-shared", "-o", out + ".tmp", *objs]):
                raise RuntimeError("hipcc failed linking the HLBM library")
            os.replace(out + ".tmp", out)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
