"""Builds the gfx950 shared library (HIP kernels + C ABI) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_NAME = "libhack_mi355x.so"
LIB_PATH = os.path.join(HERE, LIB_NAME)
STEP_CALL_PATH = os.path.join(HERE, "_step_call.so")   # CPython entry to hack_step
SOURCES = ["hack_api.cpp", "kernels_move.hip", "kernels_select.hip", "kernels_score.hip", "kernels_attn.hip", "kernels_attn_split.hip", "kernels_attn_f32.hip", "kernels_step.hip",
           "kernels_headvar.hip", "kernels_merge.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# Packed fp32 VALU forms are switched off for all device code.
# The first kernel arguments (14 SGPRs: the table and operand pointers) arrive in registers instead of through a load in
# front of everything else: most launches are latency chains of a few microseconds (schedules of 15 to 30 launches, same
# machine, without / with: one 256^2 image 96.5 / 95.4 us, 1024^2 778 / 769.5, at a tenth of the cache 534 / 524).
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-mllvm", "-amdgpu-kernarg-preload-count=16"]
# The score kernels read every MFMA result with the vector ALU straight away:
# keeping the accumulators in VGPRs spares one AGPR copy per result register.
# Its atomics come from one lane each; combined over the wave by the compiler they would be waited for where they are issued, in
# front of a barrier (score launches over 32 units, head_dim 128, 10.3 -> 9.8, 15.3 -> 14.7 us).
# The attention kernels' accumulators pass a rare branch in every stage: cut into pieces there, they no longer fit the
# registers (a launch of 568 us takes 8840).
PER_SOURCE = {"kernels_attn.hip": ["-mllvm", "-amdgpu-codegenprepare-break-large-phis=false"],
              "kernels_step.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
              "kernels_score.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form", "-mllvm", "-amdgpu-atomic-optimizer-strategy=None"]}
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option", "-Wno-inline-asm",
          "-Wno-unused-command-line-argument"]


def _compile(src: str, objdir: str, extra) -> str:
    obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON, *DEVICE_FLAGS, *PER_SOURCE.get(src, []), *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    noise = "not a recognized feature"
    msgs = [l for l in r.stderr.splitlines() if l.strip() and noise not in l and "warning generated" not in l]
    if msgs:
        sys.stderr.write("\n".join(msgs) + "\n")
    return obj


def build(verbose: bool = False, extra_flags=()) -> str:
    """Compile every source for gfx950, link libhack_mi355x.so and the CPython step entry next to this file."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, objdir, list(extra_flags)), SOURCES))
    tmp = LIB_PATH + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    tmp = STEP_CALL_PATH + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"],
           os.path.join(CSRC, "py_step.cpp"), "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for py_step.cpp:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, STEP_CALL_PATH)
    if verbose:
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])
