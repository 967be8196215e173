"""Build libsdq.so (HIP kernels for gfx950 + the host packer + the C ABI).

    python -m paper_2406_13868_amd.build        # or __graft_entry__.build()

Every source is compiled by hipcc for gfx950 only, in-tree, into
``paper_2406_13868_amd/_build/`` and linked into
``paper_2406_13868_amd/libsdq.so``, whose kernels are then checked for the
64-bit shift erratum (isa_check.py).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

try:
    from . import isa_check
except ImportError:  # run as a script
    import isa_check

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libsdq.so")

SOURCES = [
    "pack.cpp",
    "abi.hip",
    "act_quant.hip",
    "gemm_int_decode.hip",
    "gemm_int_mfma.hip",
    "gemm_int_split.hip",
    "gemm_int_small.hip",
    "gemm_mx_mfma.hip",
    "gemm_mx_small.hip",
    "gemm_mx_dense.hip",
    "gemm_dual.hip",
    "gemm_dual_decode.hip",
]

COMMON = [
    "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# Packed-fp32 VALU forms are kept out of every kernel.
HIP_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-fno-gpu-flush-denormals-to-zero"]


def hipcc() -> str:
    for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if p and os.path.exists(p):
            return p
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if src.endswith(".cpp"):
        cmd = [hipcc(), "-x", "c++", "-c", path, "-o", obj] + COMMON
    else:
        cmd = [hipcc(), "-c", path, "-o", obj] + COMMON + HIP_FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    # keep genuine warnings visible, drop the host pass note about the feature flag
    noise = "'-packed-fp32-ops' is not a recognized feature"
    msgs = [ln for ln in (r.stderr or "").splitlines() if ln.strip() and noise not in ln]
    if msgs:
        sys.stderr.write("\n".join(msgs) + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = min(len(SOURCES), max(1, (os.cpu_count() or 4)))
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-o", tmp] + objs + ["--offload-arch=gfx950", "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    if isa_check.have_tools():
        isa_check.check(tmp)
    else:
        sys.stderr.write("llvm-objdump not found: the kernels' 64-bit shifts are not checked\n")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
