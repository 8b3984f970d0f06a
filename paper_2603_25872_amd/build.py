"""Compile libdrf.so (HIP kernels + C ABI) for gfx950 and the binding's native half, in-tree."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdrf.so")
NATIVE = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))     # for this interpreter only
SOURCES = ["plan.cpp", "update.hip", "dit_kernels.hip", "gemm.hip", "gemm_wide_288.hip", "gemm_wide_256.hip", "gemm_pair.hip", "attn.hip", "attn_long.hip", "attn_short.hip", "block_chain.hip", "denoiser.hip", "calibrate.hip", "gemm_wide_192.hip", "gemm_wide_192x288.hip"]
FLAGS = ["-x", "hip", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


# Per-file extras.  Attention: keep MFMA accumulators in ordinary VGPRs; the online softmax reads
# every score right after the MFMA, and AGPR accumulators would cost one move per value per tile.
EXTRA = {name: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for name in ("attn.hip", "attn_long.hip", "attn_short.hip", "block_chain.hip")}


def _compile(src):
    out = os.path.join(OBJ, src + ".o")
    subprocess.check_call(["hipcc", *FLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", out])
    return out


def build(verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    include = sysconfig.get_paths()["include"]
    if os.path.exists(os.path.join(include, "Python.h")):
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-Wall", "-fPIC", "-shared", "-I" + include, os.path.join(CSRC, "binding.cpp"), "-o", NATIVE])
    else:
        print("no Python.h in %s: the skip calls marshal their arguments with ctypes" % include)
    if verbose:
        print("built", LIB)
    return LIB


def ensure_built():
    """For the test harness, the smoke entry and the benchmark: compile only when no library has been
    built yet.  The binding itself never builds: it raises when the library is missing."""
    if not os.path.exists(LIB):
        build(verbose=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
