"""Build libhisq.so (HIP, gfx950) in-tree with hipcc.

``python -m paper_2302_09224_amd.build`` or ``build()`` from Python.  Each
``csrc/*.hip`` file is compiled to an object under ``_build/`` (in parallel),
then linked into ``paper_2302_09224_amd/libhisq.so``.
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libhisq.so")
ARCH = os.environ.get("HISQ_OFFLOAD_ARCH", "gfx950")

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

# -packed-fp32-ops: never emit packed FP32 VALU instructions (v_pk_*_f32)
CFLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-munsafe-fp-atomics", "-ffp-contract=fast",
    # full unrolling of the stencil's hop loops also when they hold inline
    # asm (whose cost estimate would otherwise stop the unroll and leave
    # per-hop arrays indexed at run time, in scratch memory)
    "-mllvm", "-pragma-unroll-threshold=200000",
    "-Wall", "-Wno-unused-result", "-Wno-unused-command-line-argument",
    f"-I{INCLUDE}", f"-I{CSRC}",
]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    cmd = [HIPCC, *CFLAGS, "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def build(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every HIP source for gfx950 and link libhisq.so; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    # the Dslash triplets first: each takes minutes, the other sources seconds
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")), key=lambda s: ("_dslash_t_" not in s, s))
    jobs = jobs or min(len(srcs), max(1, (os.cpu_count() or 4)), 8)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
