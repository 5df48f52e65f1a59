"""Build libfa.so (the HIP kernels + C ABI) in-tree for gfx950 with hipcc.

Usage: ``python -m paper_2302_05865_amd.build``.  Cross-compiles without a GPU.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libfa.so")
# source file -> extra device-compiler flags
SOURCES = {
    "fa_kernels.hip": [],
    # matrix-core results straight into VGPRs: no accumulator-register copies in the
    # purification loop of the p x p kernel (236 -> 222 us at p = 15).  Not for the streaming
    # kernels, whose larger tilings need the accumulator registers as extra space.
    "fa_irls16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "fa_irls64.hip": [],
    "fa_gram_lp.hip": [],
    "fa_api.hip": [],
}
OBJ_DIR = os.path.join(HERE, "_build")


def hipcc_path() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError(f"hipcc failed ({proc.returncode}):\n{proc.stdout}\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)


def build(verbose: bool = True) -> str:
    common = [hipcc_path(), "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc",
              # no packed-fp32 instruction forms (some have given wrong results on this hardware)
              "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-Wall", "-Wno-unused-function"]
    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = [os.path.join(OBJ_DIR, src.replace(".hip", ".o")) for src in SOURCES]
    with ThreadPoolExecutor(len(SOURCES)) as pool:      # (one compiler a file)
        done = [pool.submit(_run, common + extra + ["-c", os.path.join(CSRC, src), "-o", obj], verbose)
                for (src, extra), obj in zip(SOURCES.items(), objs)]
        for job in done:
            job.result()
    _run([hipcc_path(), "--offload-arch=gfx950", "-fno-gpu-rdc", "-shared", "-fPIC"] + objs +
         ["-o", LIB_PATH], verbose)
    return LIB_PATH


if __name__ == "__main__":
    print(build())
