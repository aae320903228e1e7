"""Build the gfx950 shared library (paper_1808_01448_amd/_lib/liblbib.so) with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(OUT_DIR, "liblbib.so")
SOURCES = ["lbib_sweep.hip", "lbib_pool_sweep.hip", "lbib_particle.hip", "lbib_runtime.cpp", "lbib_pool.cpp",
           "lbib_serve.cpp", "lbib_host.cpp", "lbib_geometry.cpp", "lbib_static.hip",
           "lbib_fields.hip"]
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed-FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Device code is compiled without FMA contraction: the arithmetic of every kernel is then
# exactly the written sequence (with the fused operations written out where they pay), so a
# simulation gives bit-identical results whichever kernel variant runs it (one simulation
# or a pool, push or pull layout, any number of markers per thread).  The host file is built
# the same way: its equilibrium, used by read-outs of the f - f_eq storages, matches the device's.
PER_SOURCE = {src: ["-ffp-contract=off"] for src in ("lbib_sweep.hip", "lbib_pool_sweep.hip", "lbib_particle.hip", "lbib_fields.hip",
                                                        "lbib_host.cpp")}


def hipcc() -> str:
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.isabs(c) and os.path.exists(c):
            return c
    return "hipcc"


def build(verbose: bool = False) -> str:
    """Compile every source and link the library; always rebuilds."""
    os.makedirs(OUT_DIR, exist_ok=True)
    objs, cmds = [], []
    for src in SOURCES:
        obj = os.path.join(OUT_DIR, os.path.splitext(src)[0] + ".o")
        cmds.append([hipcc(), *FLAGS, *PER_SOURCE.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    procs = []
    for cmd in cmds:  # one compiler process per source, all at once
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd)))
    failed = [cmd for cmd, p in procs if p.wait() != 0]
    if failed:
        raise subprocess.CalledProcessError(1, failed[0])
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
