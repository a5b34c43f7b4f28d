"""Builds the HIP library ``liblbm_ltne.so`` for gfx950 with hipcc.

Usage: ``python -m paper_1608_04118_amd.build`` (or call ``build()``).  The
library is written next to this file so that it travels with the source tree.
"""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbm_ltne.so")
# Objects of the library: source, flags of its own.  tile.hip is compiled once
# per precision form (see there for the flag).
TILE_FLAGS = ["-mllvm", "-disable-machine-licm"]
OBJECTS = [("lbm_ltne.hip", []), ("params.hip", []), ("batch.hip", []), ("tile_shapes.hip", []),
           ("readback.hip", []), ("adjoint_tile.hip", TILE_FLAGS)]
OBJECTS += [("tile.hip", TILE_FLAGS + ["-DLTNE_TILE_FORM=%d" % form]) for form in range(4)]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # no packed-FP32 instructions in the generated device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # multiply-adds fused only within one source expression, so the node
    # update compiles to the same arithmetic in every kernel that inlines it
    # (single lattice and batch): bit-identical results by construction
    "-ffp-contract=on",
    "-Wall",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building %s" % LIB)


def build(verbose: bool = False) -> str:
    """Compile every HIP source of the library into LIB (always recompiles)."""
    work = tempfile.mkdtemp(prefix="lbm_ltne_build_")
    try:
        base = [hipcc()] + HIPCC_FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
        objs = [os.path.join(work, "%d.o" % i) for i in range(len(OBJECTS))]
        cmds = [base + flags + ["-c", "-o", obj, os.path.join(CSRC, src)]
                for obj, (src, flags) in zip(objs, OBJECTS)]
        jobs = max(1, min(len(cmds), os.cpu_count() or 1, int(os.environ.get("MAX_JOBS", "8"))))
        with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        tmp = LIB + ".tmp%d" % os.getpid()
        _run([hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, verbose)
        os.replace(tmp, LIB)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
