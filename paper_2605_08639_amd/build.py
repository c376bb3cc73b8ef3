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


def compile_source(src: str, obj: str) -> dict:
    """Compiles one source and returns what each of its kernels takes ({kernel: {"VGPRs": .., "LDS Size": .., ..}}).
    A kernel that needs scratch memory is an error: the GEMM kernels count their loads in flight by hand, and
    the reload of a spilled register, counted by the compiler, waits for all of them."""
    report = ["-Rpass-analysis=kernel-resource-usage"] if src.endswith(".hip") else []
    run = subprocess.run([HIPCC, *FLAGS, *report, "-c", src, "-o", obj], stderr=subprocess.PIPE, text=True)
    remark, kernel, usage = False, {}, {}
    for line in run.stderr.splitlines():
        if "[-Rpass-analysis=kernel-resource-usage]" in line:
            remark = True
            name = re.search(r"Function Name: (\S+)", line)
            value = re.search(r"remark:\s+([A-Za-z ]+?)(?: \[\S+\])?: (\d+) ", line)
            if name:
                kernel = usage.setdefault(name[1], {})
            elif value:
                kernel[value[1]] = int(value[2])
        elif not (remark and re.match(r"\s*\d*\s*\|", line)):      # (source excerpts follow the remarks)
            remark = False
            print(line, file=sys.stderr)
    if run.returncode:
        raise subprocess.CalledProcessError(run.returncode, run.args)
    spilled = [f"{name} ({k['ScratchSize']} bytes per lane)" for name, k in usage.items() if k["ScratchSize"]]
    if spilled:
        os.remove(obj)
        raise RuntimeError("kernels use scratch memory: " + ", ".join(spilled))
    return usage


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
