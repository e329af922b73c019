"""Build libsfrde.so in-tree for gfx950 with hipcc.

Usage: python -m paper_2003_13569_amd.build   (or build() from Python)
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "sfrde.hip")
PART = os.path.join(HERE, "csrc", "wave_part.hip")
NPARTS = 28  # classes of csrc/wave_parts.h, one translation unit each
LIB = os.path.join(HERE, "libsfrde.so")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC",
    "--offload-arch=gfx950",
    # no packed FP32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"hipcc failed with code {res.returncode}")


def build(verbose: bool = True) -> str:
    """Compile the parts (a few at a time) and link them to libsfrde.so."""
    inc = ["-I", os.path.join(ROOT, "include")]
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f"part{k}.o") for k in range(NPARTS)]
        host = os.path.join(tmp, "sfrde.o")
        cmds = [[hipcc(), *FLAGS, *inc, "-DSFRDE_IN_PARTS", "-c", SRC, "-o", host]]
        # largest classes first
        cmds += [[hipcc(), *FLAGS, *inc, f"-DSFRDE_PART={k}", "-c", PART, "-o", objs[k]]
                 for k in reversed(range(NPARTS))]
        with ThreadPoolExecutor(max(1, min(8, os.cpu_count() or 1))) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        out = LIB + ".tmp"
        _run([hipcc(), "-shared", "--offload-arch=gfx950", host, *objs, "-o", out], verbose)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
