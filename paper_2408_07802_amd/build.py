"""Builds libkraken.so (HIP, gfx950) in-tree with hipcc.

Every HIP source under csrc/ is compiled for gfx950 and linked into
``paper_2408_07802_amd/libkraken.so``.  Packed-fp32 VALU instructions are
disabled for all device code.
"""

from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libkraken.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

# (source, object name, extra flags); the large GEMM templates are compiled once per operand
# type, in parallel
SOURCES = [
    *[(f"{src}.hip", f"{src}_{t}", [f"-DKRAKEN_T={t}"])
      for src in ("gemm_tile", "gemm_mid", "gemm_skinny") for t in ("f16", "bf16", "float")],
    ("attention.hip", "attention", []), ("gemm.hip", "gemm_dispatch", []),
    ("norm.hip", "norm", []), ("decode.hip", "decode", []), ("runtime.hip", "runtime", []),
]
# one relocatable object per component (the GEMM's parts are merged into gemm.o)
OBJECTS = ["gemm", "attention", "norm", "decode", "runtime"]

COMMON_FLAGS = [
    "-std=c++17", "-O3", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Wno-unused-function",
    f"-I{os.path.join(ROOT, 'include')}",
]


# Per-file additions.  Attention: for finite inputs its softmax only takes maxima of finite
# scores and -inf; without IEEE mode the compiler drops the NaN-quieting instruction it
# otherwise puts in front of every maximum.
FILE_FLAGS = {
    "attention.hip": ["-fno-honor-nans", "-mno-amdgpu-ieee"],
}


def _compile(unit) -> str:
    src, name, extra = unit
    obj = os.path.join(BUILD_DIR, name + ".o")
    cmd = [HIPCC, *COMMON_FLAGS, *FILE_FLAGS.get(src, []), *extra, "-c",
           os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{res.stdout}\n{res.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    """Compiles every source and links the shared library; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 4)) as ex:
        list(ex.map(_compile, SOURCES))
    return link(verbose)


def link(verbose: bool = False) -> str:
    """Links the objects in BUILD_DIR into the shared library; returns its path."""
    objs = [os.path.join(BUILD_DIR, name + ".o") for name in OBJECTS]
    parts = [os.path.join(BUILD_DIR, n + ".o") for _, n, _ in SOURCES if n.startswith("gemm_")]
    res = subprocess.run(["ld", "-r", *parts, "-o", objs[0]], capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"merging the GEMM objects failed:\n{res.stdout}\n{res.stderr}")
    tmp = LIB_PATH + ".tmp"
    cmd = [HIPCC, "-shared", f"--offload-arch={ARCH}", "-fPIC", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stdout}\n{res.stderr}")
    os.replace(tmp, LIB_PATH)
    if verbose:
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
