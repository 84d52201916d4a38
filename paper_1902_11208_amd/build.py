"""Build libmdlstm.so (the C-ABI library and its HIP kernels) for gfx950, in-tree.

Usage: python -m paper_1902_11208_amd.build [--verbose]
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libmdlstm.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["mdlstm_api.cpp", "k_pack.hip", "k_proj.hip", "k_wave.hip", "k_wave_fwd_f32_h4.hip", "k_wave_fwd_f32_h8.hip",
           "k_wave_fwd_f32_h16.hip", "k_wave_fwd_f32_h32.hip", "k_wave_fwd_f32_h64.hip", "k_wave_fwd_bf16_h32.hip",
           "k_wave_fwd_bf16_h64.hip", "k_wave_bwd_f32_h4.hip", "k_wave_bwd_f32_h8.hip", "k_wave_bwd_f32_h16.hip",
           "k_wave_bwd_f32_h32.hip", "k_wave_bwd_f32_h64.hip", "k_wave_bwd_bf16_h32.hip", "k_wave_bwd_bf16_h64.hip", "k_bwd_big.hip", "k_bwd_strip.hip",
           "k_stack.hip", "k_head.hip", "k_wave_mem_h16.hip", "k_wave_mem_h32.hip", "k_pad.hip"]

FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-fPIC",
    "-std=c++17",
    "-I", INCLUDE,
    "-I", CSRC,
    # packed fp32 VALU ops stay off; the compiler otherwise forms them from scalar code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS]
    if src.endswith(".cpp"):
        cmd += ["-x", "hip"]
    cmd += ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        cmd += ["-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(ln for ln in (r.stdout + r.stderr).splitlines()
                    if "not a recognized feature" not in ln)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    if verbose and out.strip():
        print(out)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(SOURCES), max(1, min(16, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Wl,--no-undefined", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="--verbose" in sys.argv))
