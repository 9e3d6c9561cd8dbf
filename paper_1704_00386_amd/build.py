"""Build ``libnd.so`` (the HIP library behind include/nd.h) for gfx950.

Every library source in ``csrc/`` is compiled with hipcc for gfx950 only,
then linked into one shared library next to this file.  ``csrc/ceiling.hip``
(the benchmark's ceiling measurements, not part of the library) becomes
``libndceil.so`` beside it.  Usage:
``python paper_1704_00386_amd/build.py [--jobs N]`` (run as a script: importing
the package itself needs the library).
"""

from __future__ import annotations

import argparse
import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libnd.so")
CEIL_LIB = os.path.join(HERE, "libndceil.so")
CEIL_SRC = "ceiling.hip"

SOURCES = ["api.hip", "prim.hip", "graph.hip", "cliques.hip", "layout.hip",
           "sweep.hip", "tiny.hip", "driver.hip", "partial.hip", "levels.hip", "batch.hip",
           "server.hip"]

# sweep_inst.hip once per k = C(s,r) - 1 and type of tau
SWEEP_SRC = "sweep_inst.hip"
SWEEP_OBJS = [(f"sweep_k{k}_{t}", [f"-DND_SWEEP_K={k}", f"-DND_SWEEP_T={t}",
                                   f"-DND_SWEEP_BATCH={int(t != 'uint8_t')}"])
              for k in (5, 3, 2, 1) for t in ("int32_t", "uint16_t", "uint8_t")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # no packed-FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def _compile(src: str, name: str = "", defs=()) -> str:
    obj = os.path.join(OBJ, (name or os.path.splitext(src)[0]) + ".o")
    cmd = [HIPCC, *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
    # hipcc's host pass warns that it does not know the packed-fp32 feature
    return obj


def _link(objs, lib: str) -> None:
    tmp = lib + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs,
           "-o", tmp, "-lpthread", "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx",
           "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, lib)


def build(jobs: int | None = None) -> str:
    os.makedirs(OBJ, exist_ok=True)
    jobs = jobs or min(8, os.cpu_count() or 1)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        # the longest first
        lib = [ex.submit(_compile, SWEEP_SRC, n, d) for n, d in SWEEP_OBJS]
        lib += [ex.submit(_compile, s) for s in SOURCES]
        ceil = ex.submit(_compile, CEIL_SRC)
        objs, ceil_obj = [f.result() for f in lib], ceil.result()
    _link(objs, LIB)
    _link([ceil_obj], CEIL_LIB)
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=None)
    args = ap.parse_args()
    print(build(args.jobs))
    sys.exit(0)
