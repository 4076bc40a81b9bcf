"""Build libpcx.so (HIP for gfx950) in-tree with hipcc.

    python -m paper_2502_04189_amd.build        # or build() from Python
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpcx.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SOURCES = ["pcx_fft_xf.hip", "pcx_fft_xi.hip", "pcx_fft_xa.hip", "pcx_fft_yf.hip", "pcx_fft_yi.hip", "pcx_z.hip",
           "pcx_kernels.hip", "pcx_host.cpp", "pcx_batch.cpp", "pcx_tune.cpp", "pcx_noalloc.cpp",
           "flow_kernels.hip", "flow_host.cpp", "varcoef_kernels.hip", "varcoef_host.cpp"]
# kernel tables the host code refers to weakly (it also links without them):
# the library has to have them
REQUIRED = ["_ZN3pcx15fft_xfwd_kernelEii", "_ZN3pcx21fft_xinv_store_kernelEii", "_ZN3pcx21fft_xinv_accum_kernelEii",
            "_ZN3pcx15fft_yfwd_kernelEii", "_ZN3pcx15fft_yinv_kernelEii", "_ZN3pcx8z_kernelEii"]
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
         # no packed FP32 instructions anywhere in the device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    missing = [s for s in SOURCES if not os.path.exists(os.path.join(CSRC, s))]
    if missing:
        raise RuntimeError(f"sources missing from {CSRC}: {', '.join(missing)}")
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES))
    return link(objs, verbose)


def link(objs, verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    # an alias of a symbol that is not there is a link error
    cmd += [f"-Wl,--defsym=pcx_required_{i}={sym}" for i, sym in enumerate(REQUIRED)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
