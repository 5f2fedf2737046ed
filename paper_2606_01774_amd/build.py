"""Build libbdgdn.so (the HIP kernels and the C ABI) for gfx950 with hipcc.

Each source is compiled to its own object in parallel, then linked in-tree as
``paper_2606_01774_amd/libbdgdn.so``.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libbdgdn.so")
SOURCES = ["api.hip", "fwd_kernels.hip", "fwd_scan_kernels.hip", "fused_kernels.hip", "serve_kernels.hip",
           "split_kernels.hip", "conv_kernels.hip", "bwd_kernels.hip", "chunked_kernels.hip",
           "bwd_generic.hip", "bwd_steps.hip", "bwd_scan.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I" + INCLUDE, "-I" + CSRC,
         # no packed-fp32 instructions in the device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# Per-source extra flags.  The chunk-parallel and the backward scan kernels keep their MFMA accumulators in
# ordinary VGPRs (the compiler's default AGPR form copies every accumulator that VALU code
# touches in and out of the accumulation registers).
EXTRA = {"chunked_kernels.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
         "bwd_scan.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str, objdir: str) -> str:
    obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed for {src}")
    return obj


def build(verbose: bool = False) -> str:
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(lambda s: _compile(s, objdir), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libbdgdn.so failed")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
