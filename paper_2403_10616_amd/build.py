"""Compile the HIP sources under csrc/ for gfx950 into paper_2403_10616_amd/libdipaco.so (in-tree).

Usage: python -m paper_2403_10616_amd.build   (hipcc cross-compiles; no GPU needed)
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libdipaco.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # keep the compiler from forming packed fp32 ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first plain arguments of a kernel (attention, LayerNorm, routing, products of a few rows) arrive in registers instead of through a load
    # in front of everything else, 0.1 us a launch; a struct by value, as the matrix products take, is still loaded.  Without | with, us: 64 tokens
    # of the 150M path 1984 | 1957, 256 tokens of a 64-wide one 140.7 | 138.7, features of one document 327 | 320; long calls level
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
]


# per-file additions.  attention_mfma.hip (bf16, head size 64) forms no NaN of finite inputs (masked scores are -inf and every
# row keeps a finite maximum); saying so removes the canonicalising self-maxima the compiler otherwise puts in front of every
# v_max.  The kernels for the other head sizes and for fp32 honour NaN.
EXTRA_FLAGS = {"attention_mfma.hip": ["-fno-honor-nans"]}


# Kernels whose accumulators must stay in registers: a build in which the compiler moves them to scratch memory
# (it does when an unrolled loop outgrows its limits) still passes every test and runs fifteen times slower.
NO_SCRATCH = ("gemm_dlds_kernel", "gemm_fit_kernel", "gemm_fit_pair_kernel", "gemm_fit_pair_wide_kernel", "gemm_direct_kernel", "gemm_direct_pair_kernel", "gemm_direct_norm_kernel", "gemm_split_kernel", "attn_", "route_kernel", "route_small_kernel", "route_few_kernel", "sum_layernorm_kernel", "rows_product_kernel", "attn_out_kernel")


def _check_scratch(src: str, remarks: str) -> None:
    name = None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "ScratchSize [bytes/lane]:" in line and name:
            size = int(line.split("ScratchSize [bytes/lane]:")[1].split()[0])
            if size > 64 and any(k in name for k in NO_SCRATCH):   # a few spilled registers are tolerated
                raise RuntimeError(f"{os.path.basename(src)}: kernel {name} uses {size} bytes of scratch per lane")


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _up_to_date(src: str, obj: str) -> bool:
    """DIPACO_INCREMENTAL=1 (development): keep an object newer than its source, every header and this file."""
    if os.environ.get("DIPACO_INCREMENTAL") != "1" or not os.path.exists(obj):
        return False
    deps = [src, __file__] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    deps += [os.path.join(HERE, "..", "include", f) for f in os.listdir(os.path.join(HERE, "..", "include"))]
    return os.path.getmtime(obj) > max(os.path.getmtime(d) for d in deps)


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    if _up_to_date(src, obj):
        return obj
    cmd = [HIPCC, *FLAGS, *EXTRA_FLAGS.get(os.path.basename(src), []), "-Rpass-analysis=kernel-resource-usage", "-c", src,
           "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    _check_scratch(src, r.stderr)
    warn = "\n".join(l for l in r.stderr.splitlines()
                     if "packed-fp32-ops" not in l and "kernel-resource-usage" not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, sources()))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return LIB_PATH


if __name__ == "__main__":
    print(build())
