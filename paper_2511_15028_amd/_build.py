"""Builds libbvh.so (the HIP library behind include/bvh.h) for gfx950 in-tree."""
from __future__ import annotations

import concurrent.futures
import os
import re
import shutil
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(PKG, "_build")
LIB_PATH = os.path.join(PKG, "libbvh.so")
SOURCES = ["api.hip", "build.hip", "trace.hip", "closest.hip", "backward.hip", "batch.hip",
           "workspace.hip"]

HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
# -ffp-contract=off: the ray/triangle and ray/box tests must round every
# product and sum separately (no FMA contraction), like the paper's listing.
# Packed FP32 instructions are disabled for all device code.
CXXFLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-result", f"-I{INCLUDE}", f"-I{CSRC}"]


def _scratch_kernels(remarks: str) -> list:
    """Kernels whose resource-usage report (-Rpass-analysis) shows scratch
    (private) memory per lane: (name, bytes)."""
    out, name = [], None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and int(m.group(1)) > 0:
            out.append((name, int(m.group(1))))
    return out


# Persistent kernels hold four waves per SIMD, what their LDS allows (512
# registers a lane of a SIMD), and wait for memory: one wave fewer costs up to
# a quarter.
MAX_VGPRS = 128
PERSISTENT = ("k_trace_persist", "k_batch_trace", "k_cpq_persist")


def _large_kernels(remarks: str) -> list:
    """Persistent kernels whose report shows more registers than that:
    (name, registers)."""
    out, name = [], None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"\bVGPRs: (\d+)", line)
        if m and int(m.group(1)) > MAX_VGPRS and any(k in (name or "") for k in PERSISTENT):
            out.append((name, int(m.group(1))))
    return out


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CXXFLAGS, "-Rpass-analysis=kernel-resource-usage", "-c",
           os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
    # no kernel may use scratch memory: the runtime sizes a scratch
    # allocation for every resident wave around each launch that needs it
    bad = _scratch_kernels(r.stderr)
    if bad:
        raise RuntimeError(f"{src}: kernels using scratch memory: {bad}")
    large = _large_kernels(r.stderr)
    if large:
        raise RuntimeError(f"{src}: persistent kernels of more than {MAX_VGPRS} registers: {large}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB_PATH + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB_PATH)
    if verbose:
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build(verbose=True)
