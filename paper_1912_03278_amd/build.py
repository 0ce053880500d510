"""Build the HIP library libihmc.so for gfx950 (in-tree, next to this file).

    python -m paper_1912_03278_amd.build

Every source under csrc/ is compiled by hipcc on its own (in parallel) and the
objects are linked into one library.  Flags:
  * --offload-arch=gfx950                 MI355X (CDNA4)
  * -ffp-contract=off                     arithmetic exactly as written (explicit fma only),
                                          so every kernel computes a site bit-identically
  * -target-feature -packed-fp32-ops      no packed FP32 instructions
and per source, PER_SOURCE:
  * -disable-machine-licm (resident_kernels.hip): the trajectory loop holds the FP64 draws and action
    terms, whose ~60 polynomial constants the compiler otherwise keeps in registers across the whole
    loop, spilling the site state (fp32 2D, four sites a thread: 340 -> 0 bytes of scratch at 128 VGPRs)
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libihmc.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-Xclang", "-target-feature",
         "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         "-I", os.path.join(HERE, "..", "include")]
PER_SOURCE = {"resident_kernels.hip": ["-mllvm", "-disable-machine-licm"]}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed")


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        objs = []
        jobs = []
        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            for src in sources():
                name = os.path.basename(src)
                obj = os.path.join(d, name + ".o")
                objs.append(obj)
                jobs.append(pool.submit(_run, [HIPCC, *FLAGS, *PER_SOURCE.get(name, []), "-c", src, "-o", obj], verbose))
            for j in jobs:
                j.result()
        _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
