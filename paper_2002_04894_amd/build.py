"""Builds the gfx950 HIP library `libfmm.so` in-tree with hipcc.

Usage: python -m paper_2002_04894_amd.build   (or build() from Python)
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfmm.so")
BUILD_DIR = os.path.join(HERE, "_build")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    # never let the compiler emit packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
    "-Wall", "-Wno-unused-function", "-Wno-unused-result",
]


# sources compiled in several parts (-DFMM_PART=0, 1, ...), each a unit of its own
PARTS = {"m2l_quad.hip": 4}


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def units():
    """(source, part or None), those in parts first: they take longest."""
    out = []
    for src in sources():
        out += [(src, k) for k in range(PARTS.get(os.path.basename(src), 0))] or [(src, None)]
    return sorted(out, key=lambda u: u[1] is None)


def _compile(unit) -> str:
    src, part = unit
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ("" if part is None else f".{part}") + ".o")
    cmd = [HIPCC, *FLAGS, *([] if part is None else [f"-DFMM_PART={part}"]), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "not a recognized feature" not in l
                    and "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{out}")
    if out.strip():
        print(out, file=sys.stderr)
    return obj


def build(verbose: bool = True) -> str:
    """Compile every HIP source for gfx950 and link libfmm.so (always rebuilds)."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    todo = units()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(todo))) as ex:
        objs = list(ex.map(_compile, todo))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, OUT)
    if verbose:
        print(f"built {OUT}")
    return OUT


if __name__ == "__main__":
    build()
