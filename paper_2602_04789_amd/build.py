"""Compile the C-ABI library ``liblf_hsa.so`` for gfx950 with hipcc (in-tree).

    python -m paper_2602_04789_amd.build

hipcc cross-compiles without a GPU.  Device code is built with packed-FP32 VALU ops
disabled; the host file is built with -ffp-contract=off because the budget arithmetic
must round exactly as written.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "liblf_hsa.so")
BENCH_LIB = os.path.join(PKG, "liblf_bench.so")
PROBES = ("none", "tr", "k", "mfma", "exp")


def probe_lib(tag: str) -> str:
    return os.path.join(PKG, f"liblf_hsa_probe_{tag}.so")
OBJ = os.path.join(PKG, "_build")

SOURCES = ["lf_host.cpp", "lf_select.hip", "lf_attn.hip", "lf_attn_wide.hip", "lf_attn_bwd.hip", "lf_attn_bwd_wide.hip", "lf_attn_bwd_q_wide.hip",
           "lf_producer.hip"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-Wall", "-Wno-unused-function"]
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          # keep MFMA accumulators in ordinary VGPRs (the attention kernel's softmax reads
          # them with vector-ALU instructions; the AGPR form costs a copy around every use)
          "-mllvm", "-amdgpu-mfma-vgpr-form=1"]
# Per-file additions.  The attention kernel produces no NaN from finite inputs (its masks
# are -inf and its running maximum starts finite), so max() there need not quiet signalling
# NaNs first: that drops one vector instruction per score.  The selection kernels keep the
# default: their comparisons define the bit-exact index lists.  The scheduling strategy is the
# one that measured fastest for this kernel (1-2 % over the default on three workloads).
PER_FILE = {"lf_attn.hip": ["-fno-honor-nans", "-mllvm", "-amdgpu-sched-strategy=max-memory-clause"],
            "lf_attn_wide.hip": ["-fno-honor-nans"]}


def _hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found (need ROCm)")
    return exe


def _run(cmd):
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout)
        raise RuntimeError("build failed: " + " ".join(cmd))
    return res.stdout


def build(verbose: bool = False, extra_device_flags=()) -> str:
    hipcc = _hipcc()
    os.makedirs(OBJ, exist_ok=True)
    objs = []
    for src in SOURCES:
        path = os.path.join(CSRC, src)
        obj = os.path.join(OBJ, src.replace(".", "_") + ".o")
        if src.endswith(".hip"):
            cmd = ([hipcc, "-c", path, "-o", obj] + COMMON + DEVICE + PER_FILE.get(src, []) +
                   list(extra_device_flags))
        else:
            cmd = [hipcc, "-x", "c++", "-c", path, "-o", obj, "-ffp-contract=off"] + COMMON
        out = _run(cmd)
        if verbose and out.strip():
            print(out)
        objs.append(obj)
    _run([hipcc, "-shared", "-o", LIB] + objs + ["--offload-arch=gfx950"])
    # probe builds of the library for `bench.py --sensitivity`: the attention kernel with redundant
    # work per step for one unit each (LF_PROBE_*; none: without), everything else the same objects
    for tag in PROBES:
        pobj = os.path.join(OBJ, f"lf_attn_probe_{tag}_hip.o")
        _run([hipcc, "-c", os.path.join(CSRC, "lf_attn.hip"), "-o", pobj, "-DLF_PROBE", f"-DLF_PROBE_{tag.upper()}"] +
             COMMON + DEVICE + PER_FILE["lf_attn.hip"])
        _run([hipcc, "-shared", "-o", probe_lib(tag)] + [o for o in objs if os.path.basename(o) != "lf_attn_hip.o"] + [pobj] +
             ["--offload-arch=gfx950"])
    # probe build for `bench.py --select-phases`: the selection kernel with wall-clock stamps at its
    # phase boundaries (LF_PROBE_STAMPS), everything else the same objects
    sobj = os.path.join(OBJ, "lf_select_probe_stamps_hip.o")
    _run([hipcc, "-c", os.path.join(CSRC, "lf_select.hip"), "-o", sobj, "-DLF_PROBE_STAMPS"] + COMMON + DEVICE)
    _run([hipcc, "-shared", "-o", probe_lib("stamps")] + [o for o in objs if os.path.basename(o) != "lf_select_hip.o"] +
         [sobj] + ["--offload-arch=gfx950"])
    # the benchmark's micro-benchmarks: a library of their own, not linked into the product
    bobj = os.path.join(OBJ, "lf_bench_hip.o")
    _run([hipcc, "-c", os.path.join(CSRC, "lf_bench.hip"), "-o", bobj] + COMMON + DEVICE)
    _run([hipcc, "-shared", "-o", BENCH_LIB, bobj, "--offload-arch=gfx950"])
    return LIB


def build_sanitized_host(out_dir: str = OBJ) -> str:
    """Host side of the C ABI alone (lf_host.cpp: validation, budgets, sizes) compiled for the CPU
    with AddressSanitizer and UndefinedBehaviorSanitizer, linked with the test driver that stands
    in for the kernel launchers.  Returns the executable's path; no GPU code is involved."""
    gxx = shutil.which("g++")
    if not gxx:
        raise RuntimeError("g++ not found")
    os.makedirs(out_dir, exist_ok=True)
    exe = os.path.join(out_dir, "lf_host_sanitized")
    _run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
          "-fno-omit-frame-pointer", "-ffp-contract=off", "-Wall", "-I", os.path.join(ROOT, "include"),
          "-I", CSRC, os.path.join(CSRC, "lf_host.cpp"),
          os.path.join(ROOT, "tests", "host_sanitize_driver.cpp"), "-o", exe])
    return exe


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
    if "--sanitize" in sys.argv:
        print(build_sanitized_host())
