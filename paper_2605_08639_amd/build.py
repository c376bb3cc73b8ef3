"""Builds librelibra.so (HIP kernels + host planner) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librelibra.so")
SOURCES = ["route_kernels.hip", "ffn_kernels.hip", "replica_kernels.hip", "prof.hip", "plan.cpp", "reorder_sa.cpp", "split.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # loop heads on 32-byte boundaries: the batched weight-gradient k-loop measured 6 % slower when a
         # change elsewhere in the file moved it to an unaligned address
         "-falign-loops=32",
         "-Wall", "-Wno-unused-function"]


def compile_source(src: str, obj: str) -> None:
    """Compiles one source.  A kernel that needs scratch memory is an error: the GEMM kernels count their loads in
    flight by hand, and the reload of a spilled register, counted by the compiler, waits for all of them."""
    report = ["-Rpass-analysis=kernel-resource-usage"] if src.endswith(".hip") else []
    run = subprocess.run([HIPCC, *FLAGS, *report, "-c", src, "-o", obj], stderr=subprocess.PIPE, text=True)
    remark, name, spilled = False, "", []
    for line in run.stderr.splitlines():
        if "[-Rpass-analysis=kernel-resource-usage]" in line:
            remark = True
            found = re.search(r"(Function Name|ScratchSize \[bytes/lane\]): (\S+)", line)
            if found and found[1] == "Function Name":
                name = found[2]
            elif found and found[2] != "0":
                spilled.append(f"{name} ({found[2]} bytes per lane)")
        elif not (remark and re.match(r"\s*\d*\s*\|", line)):      # (source excerpts follow the remarks)
            remark = False
            print(line, file=sys.stderr)
    if run.returncode:
        raise subprocess.CalledProcessError(run.returncode, run.args)
    if spilled:
        os.remove(obj)
        raise RuntimeError("kernels use scratch memory: " + ", ".join(spilled))


def build(verbose: bool = False) -> str:
    objs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        if verbose:
            print(" ".join([HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]), flush=True)
        compile_source(os.path.join(CSRC, src), obj)
        objs.append(obj)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs, "-lpthread"]
    if verbose:
        print(" ".join(cmd))
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
