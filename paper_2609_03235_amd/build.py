"""Build libsgdkv.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

Every HIP source is compiled with packed FP32 instructions disabled. The host
file is compiled without FP contraction, because the budget allocation's fp64
arithmetic decides integers and must happen in the order written.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libsgdkv.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-command-line-argument"]
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# The scheduler that puts instruction parallelism first, for the instances of the score passes that
# measured faster with it (lse_pass.h, colsum_pass.h).
ILP = ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]
FILE_FLAGS = {"lse_kernels_ilp.hip": ILP, "score_kernels_ilp.hip": ILP}
KERNEL_SOURCES = ["lse_kernels.hip", "lse_kernels_ilp.hip", "score_kernels.hip", "score_kernels_ilp.hip",
                  "select_kernels.hip", "decode_kernels.hip", "decode_scratch.hip"]
HOST_SOURCES = ["sgdkv_host.cpp", "profile.cpp"]


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l and "(ignoring feature)" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"command failed: {' '.join(cmd)}\n{err}")
    return err


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    jobs = []
    for src in KERNEL_SOURCES:
        obj = os.path.join(BUILD_DIR, src.replace(".hip", ".o"))
        jobs.append([HIPCC, *COMMON, *DEVICE, *FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj])
    for src in HOST_SOURCES:
        obj = os.path.join(BUILD_DIR, src.replace(".cpp", ".o"))
        jobs.append([HIPCC, *COMMON, "-ffp-contract=off", "-fno-fast-math", "-x", "c++", "-D__HIP_PLATFORM_AMD__",
                     "-isystem", "/opt/rocm/include",
                     "-c", os.path.join(CSRC, src), "-o", obj])
    workers = min(len(jobs), int(os.environ.get("MAX_JOBS", "8")))
    with concurrent.futures.ThreadPoolExecutor(max_workers=workers) as ex:
        for err in ex.map(_run, jobs):
            if verbose and err.strip():
                print(err, file=sys.stderr)
    objs = [j[j.index("-o") + 1] for j in jobs]
    tmp = LIB_PATH + ".tmp"
    _run([HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
