"""Build libdbsp.so (HIP, gfx950 only) in-tree with hipcc."""

from __future__ import annotations

import os
import shutil
import subprocess

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libdbsp.so")

SOURCES = ["planner.cpp", "dual_balance.cpp", "cost_model.cpp", "api.hip", "attn_fwd.hip", "mfma_probe.hip"]

# Per-file extra flags.  The attention kernels never rely on NaN propagation; without NaN
# handling the max chains of the softmax compile to v_max3_f32.  (Host-side argument checks in
# api.hip do test for NaN, so the flag is not global.)  The ILP-driven machine scheduler
# interleaves the softmax's vector work with the MFMAs better than the default one (measured).
# VGPR-form MFMAs: the 512-register instances would otherwise form every product in accumulation
# registers and copy the scores out of them one by one.
# The host planners' loops are fast or slow by where they begin: functions begin at multiples of 64 bytes, so that a change
# elsewhere does not move them (partition of 26 heads, 78 x 78 blocks: 29.4 us, 30.8 with all code 32 bytes on).
HOST_LAYOUT = ["-falign-functions=64"]
EXTRA_FLAGS = {"planner.cpp": HOST_LAYOUT, "dual_balance.cpp": HOST_LAYOUT, "attn_fwd.hip": ["-fno-honor-nans", "-mllvm", "-amdgpu-sched-strategy=iterative-ilp", "-mllvm", "-amdgpu-mfma-vgpr-form"]}

# Packed-FP32 VALU ops are switched off for all device code (-packed-fp32-ops removes the feature).
HIP_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (set HIPCC or install ROCm under /opt/rocm)")


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source and link libdbsp.so next to this file.  Always recompiles."""
    hipcc = _hipcc()
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + HIP_FLAGS + EXTRA_FLAGS.get(src, []) + list(extra_flags) + inc
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    tmp = LIB_PATH + ".tmp"
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}")
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
