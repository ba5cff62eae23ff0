"""Builds libmpcr.so (gfx950) in the package directory from csrc/.

    python -m paper_2406_02701_amd.build

Each source is compiled by hipcc into _build/ (in parallel) and linked into
paper_2406_02701_amd/libmpcr.so.  The build always recompiles.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libmpcr.so")
INCLUDE = os.path.join(os.path.dirname(PKG), "include")

ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17", "-Wall", "-Wno-unused-function",
    "-Wno-unused-variable", "-Wno-unknown-pragmas",
    # keep the compiler from forming packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    f"-I{INCLUDE}",
]
# roctx ranges (rocprofiler-sdk)
LINK_FLAGS = ["-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx"]
# the factorisation's kernels: three sources compiled side by side (the slowest of
# the library), joined into the one object factor.o
FACTOR_PARTS = ["update.hip", "factor.hip", "panel.hip"]
SOURCES = FACTOR_PARTS + ["tiles.hip", "solve.hip", "order.hip", "gemm.hip", "laplace.hip", "mala.hip",
                          "krylov.hip", "api.cpp", "serve.cpp"]


def _compile(src: str) -> str:
    stem = os.path.splitext(src)[0]
    obj = os.path.join(BUILD, stem + (".part.o" if src in FACTOR_PARTS else ".o"))
    cmd = [HIPCC, *CFLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _linker() -> str:
    """The linker that joins relocatable objects: LD_LLD, else ROCm's, else the system's."""
    names = [os.environ["LD_LLD"]] if "LD_LLD" in os.environ else ["/opt/rocm/llvm/bin/ld.lld", "ld.lld", "ld"]
    for name in names:
        if shutil.which(name):
            return name
    raise RuntimeError(f"linker not found: {', '.join(names)}")


def _link(cmd: list) -> None:
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")


def build(jobs: int = 8) -> str:
    if not shutil.which(HIPCC) and not os.path.exists(HIPCC):
        raise RuntimeError("hipcc not found")
    ld = _linker()
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    parts, objs = objs[:len(FACTOR_PARTS)], objs[len(FACTOR_PARTS):]
    factor = os.path.join(BUILD, "factor.o")
    _link([ld, "-r", *parts, "-o", factor])
    tmp = LIB + ".tmp"
    _link([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", factor, *objs, *LINK_FLAGS, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
