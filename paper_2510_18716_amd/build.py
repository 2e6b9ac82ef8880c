"""Compile the HIP sources under csrc/ into libssd_hip.so (gfx950 only), in tree.

Run as `python paper_2510_18716_amd/build.py` (not with -m: importing the package loads the library); __graft_entry__.build() calls build(force=True).
Every source is compiled to an object file of its own (in parallel, under csrc/_build/), then linked.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(HERE, "libssd_hip.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed-fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def headers():
    return sorted(glob.glob(os.path.join(CSRC, "*.h"))) + sorted(glob.glob(os.path.join(ROOT, "include", "*.h")))


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(p) > t for p in sources() + headers())


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        sys.stderr.write(r.stdout)
        raise RuntimeError("hipcc failed: " + " ".join(cmd))
    if verbose and out.strip():
        print(out)


def build(force: bool = False, verbose: bool = True) -> str:
    """force: recompile every source; otherwise only sources newer than their object (or older than a header)."""
    if not force and not is_stale():
        return LIB
    os.makedirs(OBJ, exist_ok=True)
    t_hdr = max(os.path.getmtime(p) for p in headers())
    jobs, objs = [], []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        part_of = os.path.join(CSRC, "ssd_step.hip") if os.path.basename(src).startswith("ssd_step_") else src     # included
        if force or not os.path.exists(obj) or os.path.getmtime(obj) < max(os.path.getmtime(src), os.path.getmtime(part_of), t_hdr):
            jobs.append([HIPCC] + FLAGS + ["-c", src, "-o", obj])
    jobs.sort(key=lambda c: "ssd_step_" not in c[-1])                # the longest first
    with ThreadPoolExecutor(max(1, min(8, len(jobs)))) as ex:
        list(ex.map(lambda c: _run(c, verbose), jobs))
    tmp = LIB + ".tmp%d" % os.getpid()
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(force="--incremental" not in sys.argv)
