"""Builds libspecverify.so (all HIP sources, gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
SO = os.path.join(HERE, "libspecverify.so")
# (source, object, flags): the GEMM's kernels are compiled one per object, which is most of the build's time
SOURCES = [(f + ".hip", f + ".o", []) for f in ("engine", "kernels_basic", "kernels_state", "kernels_accept", "gemm_mfma",
                                                "attn_mfma", "planner")]
SOURCES += [("gemm_mfma.hip", "gemm_mfma_%d.o" % i, ["-DSV_GEMM_PART=%d" % i]) for i in range(1, 15)]
# packed-fp32 instruction forms are disabled on purpose (they have produced wrong results on this
# hardware pool); hipcc's host pass prints a harmless "unknown feature" warning for the flag.
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def _stale(out, deps):
    return not os.path.exists(out) or any(os.path.getmtime(d) > os.path.getmtime(out) for d in deps)


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hdrs = [os.path.join(CSRC, "common.h"), os.path.join(HERE, "..", "include", "specverify.h")]
    jobs = []
    for src, obj, flags in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, obj)
        if force or _stale(o, [s] + hdrs):
            jobs.append(["hipcc", *FLAGS, *flags, "-c", s, "-o", o])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed: " + " ".join(cmd))
        return r

    with ThreadPoolExecutor(max_workers=8) as ex:
        list(ex.map(run, jobs))
    objs = [os.path.join(OBJ, o) for _, o, _ in SOURCES]
    if force or jobs or _stale(SO, objs):
        run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", SO, *objs])
    return SO


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
