"""Compile the HIP library for gfx950 into paper_2608_16329_amd/libmlip.so.

Every source is compiled by hipcc as HIP (objects in _build/, in parallel),
then linked into one shared library.  Flags: -O3, float64 atomics as
hardware atomics (-munsafe-fp-atomics), and packed-fp32 instruction
selection disabled.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmlip.so")
ARCH = "gfx950"
# The fused kernel's matrix sums are read by vector instructions right away:
# kept in vector registers they need no copies (the compiler's default for a
# kernel of 512 registers is the accumulation file).
VGPR_SUMS = ["-mllvm", "-amdgpu-mfma-vgpr-form"]
# (source, object, further flags); the fused kernel's instantiations are built
# in six parts
SOURCES = [("api.cpp", "api", []), ("angular_tables.cpp", "angular_tables", []), ("neighbors.hip", "neighbors", []),
           ("fused.hip", "fused_f64_digits", ["-DMLIP_FUSED_PART=1", "-DMLIP_FUSED_DIGITS=1"] + VGPR_SUMS),
           ("fused.hip", "fused_f64_high_digits", ["-DMLIP_FUSED_PART=2", "-DMLIP_FUSED_DIGITS=1"] + VGPR_SUMS),
           ("fused.hip", "fused_f32_digits", ["-DMLIP_FUSED_PART=3", "-DMLIP_FUSED_DIGITS=1"]),
           ("fused.hip", "fused_f64_float", ["-DMLIP_FUSED_PART=1", "-DMLIP_FUSED_DIGITS=0"]),
           ("fused.hip", "fused_f64_high_float", ["-DMLIP_FUSED_PART=2", "-DMLIP_FUSED_DIGITS=0"]),
           ("fused.hip", "fused_f32_float", ["-DMLIP_FUSED_PART=3", "-DMLIP_FUSED_DIGITS=0"]),
           ("pack.hip", "pack", []), ("unfused.hip", "unfused", []), ("md.hip", "md", []), ("scratch.hip", "scratch", [])]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def common_flags():
    return ["-x", "hip", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function"]


def _compile(entry) -> str:
    src, name, flags = entry
    obj = os.path.join(BUILD, name + ".o")
    cmd = [hipcc()] + common_flags() + flags + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    warn = [l for l in res.stderr.splitlines() if "warning" in l and "packed-fp32" not in l]
    if warn:
        sys.stderr.write("\n".join(warn) + "\n")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
