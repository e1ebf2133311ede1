"""Build libabft.so (the HIP kernels and the C ABI) for gfx950, in-tree.

    python -m paper_2104_09455_amd.build        # or: from paper_2104_09455_amd.build import build

Each .hip file under csrc/ is compiled to an object in parallel, then linked into
paper_2104_09455_amd/libabft.so.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libabft.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # keep the compiler from emitting packed-fp32 VALU forms
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
FLAGS += os.environ.get("ABFT_EXTRA_HIPCC_FLAGS", "").split()   # e.g. -D switches of tuning experiments
# (the ones that take longest first)
SOURCES = [f"gemm_{family}_{dt}.hip" for family in ("fast", "generic", "stream", "group") for dt in ("f16", "bf16", "i8")]
SOURCES += ["gemm_strip_f16.hip", "gemm_strip_bf16.hip", "abft_api.hip"] + [f"gemm_skinny_{dt}.hip" for dt in ("f16", "bf16", "i8")]


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
