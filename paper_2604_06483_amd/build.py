"""Builds the HIP library for gfx950 in-tree: paper_2604_06483_amd/libll.so.

    python -m paper_2604_06483_amd.build

hipcc cross-compiles without a GPU.  The packed-fp32 instructions are switched off for all
device code.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = ["ll_api.hip", "ll_project.hip", "ll_project_tail.hip", "ll_project_short.hip", "ll_project_sweep.hip", "ll_steer.hip", "ll_capture.hip"]
LIB = os.path.join(HERE, "libll.so")
OBJ_DIR = os.path.join(HERE, "_build")   # (git-ignored)

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
]


def build(verbose: bool = True, extra_flags=()) -> str:
    """Compiles the sources side by side and links them."""
    def run(cmds):
        if verbose:
            print("\n".join(" ".join(c) for c in cmds), flush=True)
        procs = [subprocess.Popen(c, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True) for c in cmds]
        outs = [p.communicate()[0] for p in procs]
        for p, out in zip(procs, outs):
            if p.returncode != 0:
                raise RuntimeError(f"hipcc failed ({p.returncode}):\n{out}")
            # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless noise.
            err = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
            if verbose and err.strip():
                print(err, file=sys.stderr)

    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = [os.path.join(OBJ_DIR, s.replace(".hip", ".o")) for s in SOURCES]
    run([["hipcc", *FLAGS, *extra_flags, "-c", os.path.join(HERE, "csrc", s), "-o", o] for s, o in zip(SOURCES, objs)])
    run([["hipcc", *FLAGS, "-shared", *objs, "-o", LIB]])
    return LIB


if __name__ == "__main__":
    build(extra_flags=sys.argv[1:])
    print("built", LIB)
