"""Build libpsd.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "lib", "libpsd.so")
SOURCES = ["psd_race.hip", "psd_mpfr.hip", "psd_topk.hip", "psd_gen.hip", "psd_detect.hip", "psd_api.cpp"]
ARCH = "gfx950"
# Packed-fp32 VALU forms are kept out of every kernel.
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]
# The kernels that read logits treat NaN as undefined input, so a float max needs no NaN
# quieting (which costs an instruction per loaded value in the streaming passes).
# The race kernel's LDS atomics (the best score, list counters) are issued as they are:
# the default atomic optimizer turns a same-address atomic with per-lane values into a scalar
# loop over the active lanes (about 70 cycles per lane), far slower than the LDS
# serialising the lanes' atomics itself.
EXTRA = {"psd_race.hip": ["-fno-honor-nans", "-mllvm", "-amdgpu-atomic-optimizer-strategy=None"],
         "psd_mpfr.hip": ["-fno-honor-nans"], "psd_topk.hip": ["-fno-honor-nans"],
         "psd_gen.hip": ["-ffp-contract=off"]}


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = [hipcc()] + FLAGS + EXTRA.get(src, []) + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compile every HIP source and link lib/libpsd.so (always recompiles)."""
    os.makedirs(BUILD, exist_ok=True)
    os.makedirs(os.path.dirname(LIB), exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


def build_test_helper(src: str) -> str:
    """Compile one HIP source of the tests to lib<name>.so in the _build folder beside it."""
    out = os.path.join(os.path.dirname(src), "_build", "lib" + os.path.splitext(os.path.basename(src))[0] + ".so")
    os.makedirs(os.path.dirname(out), exist_ok=True)
    r = subprocess.run([hipcc()] + FLAGS + ["-shared", src, "-o", out], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return out


if __name__ == "__main__":
    build(verbose=True)
