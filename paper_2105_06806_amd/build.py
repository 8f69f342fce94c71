"""Build libedx.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2105_06806_amd.build [--jobs N] [--debug]

Every translation unit under csrc/ is compiled for gfx950 only and linked into
paper_2105_06806_amd/libedx.so next to this file.  Packed FP32 instructions are
disabled (-packed-fp32-ops) for every device compile.
"""
from __future__ import annotations

import argparse
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libedx.so")
BUILD = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

COMMON = [
    "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    "-mcode-object-version=5",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
]


# hv.hip holds a few hundred kernel instances: it is compiled in pieces (see
# EDX_HV_PART there), the pieces first since they take longest
PARTS = {"hv.hip": 6}


def sources():
    """(source, piece or None) of every translation unit."""
    files = sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))
    pieces = [(os.path.join(CSRC, f), k) for f in files for k in range(PARTS.get(f, 0))]
    return pieces + [(os.path.join(CSRC, f), None) for f in files]


def _compile(unit, debug):
    src, part = unit
    name = os.path.basename(src) + ("" if part is None else f".{part}")
    obj = os.path.join(BUILD, name + ".o")
    cmd = [HIPCC, "-x", "hip", "-c", src, "-o", obj] + COMMON + (["-O1", "-g"] if debug else ["-O3"])
    if part is not None:
        cmd.append(f"-DEDX_HV_PART={part}")
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(jobs=None, debug=False, verbose=True):
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    jobs = jobs or min(8, os.cpu_count() or 4, len(srcs))
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, debug), srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-o", tmp] + objs + [f"--offload-arch={ARCH}", "-fPIC"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} from {len(srcs)} sources", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=None)
    ap.add_argument("--debug", action="store_true")
    a = ap.parse_args()
    build(a.jobs, a.debug)
