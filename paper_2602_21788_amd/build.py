"""Builds libfcp.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2602_21788_amd.build [--force]
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libfcp.so")
SOURCES = ["fcp_host.cpp", "fcp_planner.cpp", "fcp_sched.hip", "fcp_rowops.hip", "fcp_attn_fwd.hip", "fcp_attn_fwd_small.hip", "fcp_attn_bwd_lists.hip", "fcp_attn_bwd.hip", "fcp_attn_bwd_fused.hip", "fcp_attn_bwd_short.hip"]
HEADERS = [os.path.join(CSRC, "fcp_internal.h"), os.path.join(CSRC, "fcp_sizes.h"), os.path.join(CSRC, "fcp_device.h"), os.path.join(CSRC, "fcp_items.h"), os.path.join(CSRC, "fcp_bwd.h"), os.path.join(CSRC, "fcp_fwd.h"),
           os.path.join(ROOT, "include", "fcp.h")]
# packed fp32 VALU ops are switched off for all device code (see the note in the package docs)
# Loops begin on a cache line: a step loop is entered some thousand times by each of a block's waves and fits a step of 1000 to 3000 clocks, and
# where the compiler happens to put it moves the backward's D = 64 kernels by 2 to 5 % (20 packed sequences of 12000 tokens, 64 query heads on
# 8 KV heads: backward 1304 us at one place, 1250 us aligned).
FLAGS = ["-O3", "-falign-loops=64", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _stale(out: str, deps) -> bool:
    if not os.path.exists(out):
        return True
    t = os.path.getmtime(out)
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()
    flags = FLAGS
    jobs = []
    for src in SOURCES:
        sp = os.path.join(CSRC, src)
        op = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
        if force or _stale(op, [sp] + HEADERS):
            jobs.append([hipcc] + flags + ["-c", sp, "-o", op])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + r.stdout + r.stderr)
        return r.stderr

    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        for err in ex.map(run, jobs):
            if verbose and err:
                print(err)
    objs = [os.path.join(OBJ, os.path.splitext(s)[0] + ".o") for s in SOURCES]
    if force or jobs or _stale(LIB, objs):
        run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
