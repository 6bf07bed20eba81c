"""Build libbsa.so (HIP for gfx950) in-tree with hipcc.

Usage: python paper_2609_25869_amd/build.py [--jobs N]

Run it as a script: importing it through the package would import the
package, which refuses to load before libbsa.so exists.
"""
from __future__ import annotations

import argparse
import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbsa.so")

SOURCES = ["runtime.hip", "plan_kernels.hip", "attn_fwd.hip", "sparsify.hip", "task_order.hip", "catalog.cpp"]
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libbsa.so)")


def common_flags():
    return ["-O3", "-std=c++17", "-fPIC", "--offload-arch=%s" % ARCH,
            # keep packed-fp32 instructions out of the generated code
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-result",
            # export only the C-ABI (declared BSA_API in bsa.h)
            "-fvisibility=hidden"]


# Per-file flags.  The score tiles are VALU operands, so MFMA results stay in
# VGPRs; the compiler's default for kernels with one wave per SIMD is AGPRs,
# from which every score element would first be copied.  No flag may let the
# compiler assume that there is no NaN: the attention kernel masks through the
# addend of the exponent and finds masked scores that are not finite by the
# NaN they give.
EXTRA_FLAGS = {"attn_fwd.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
               "sparsify.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [hipcc()] + common_flags() + EXTRA_FLAGS.get(src, []) + (["-x", "c++"] if src.endswith(".cpp") else []) + \
        ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature; that warning is expected
    msgs = [l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and "warning generated" not in l
            and "warnings generated" not in l]
    if r.returncode != 0:
        raise RuntimeError("compiling %s failed:\n%s" % (src, "\n".join(msgs)))
    if msgs:
        sys.stderr.write("\n".join(msgs) + "\n")
    return obj


def build(jobs: int = 4, verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=max(1, jobs)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=%s" % ARCH] + objs + ["-o", tmp, "-ldl"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("linking libbsa.so failed:\n" + r.stdout)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=4)
    a = ap.parse_args()
    build(a.jobs, verbose=True)


if __name__ == "__main__":
    main()
