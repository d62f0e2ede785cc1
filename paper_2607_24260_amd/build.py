"""Build libkap.so (the HIP kernels and the kap.h C ABI) for gfx950, in-tree.

    python -m paper_2607_24260_amd.build

Each .hip source is compiled to an object in parallel, then linked into
paper_2607_24260_amd/libkap.so. Every HIP source is compiled with packed
FP32 instructions disabled. The build fails when a kernel of a source in
NO_SPILLS spills vector registers or takes scratch memory.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import re
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libkap.so")

ARCH = "gfx950"
HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    f"-I{INCLUDE}", f"-I{CSRC}",
]

# Sources whose kernels must hold everything in registers: versions of the wide
# attention kernel that spilled vector registers have returned wrong results.
NO_SPILLS = {"attn_wide.hip"}
RESOURCE_REMARKS = "-Rpass-analysis=kernel-resource-usage"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libkap)")


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def spills(remarks: str):
    """(kernel, spilled vector registers, scratch bytes per lane) of the kernels
    in the compiler's resource remarks that have either."""
    found, kernel, scratch = [], None, 0
    for line in remarks.splitlines():
        m = re.search(r"(Function Name|ScratchSize \[bytes/lane\]|VGPRs Spill): (\S+)", line)
        if not m:
            continue
        if m[1] == "Function Name":
            kernel = m[2]
        elif m[1].startswith("Scratch"):
            scratch = int(m[2])
        elif int(m[2]) or scratch:
            found.append((kernel, int(m[2]), scratch))
    return found


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.basename(src)[:-4] + ".o")
    checked = os.path.basename(src) in NO_SPILLS
    cmd = [hipcc(), *HIPCC_FLAGS, *([RESOURCE_REMARKS] if checked else []), "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msgs}")
    if checked:
        if "VGPRs Spill" not in msgs:
            raise RuntimeError(f"no resource remarks for {src}: its spills are unknown")
        if spills(msgs):
            raise RuntimeError(f"{src} spills (kernel, registers, scratch bytes): {spills(msgs)}")
        msgs = ""
    if verbose and msgs.strip():
        print(msgs, flush=True)
    return obj


def build(verbose: bool = False) -> str:
    """Compile every HIP source for gfx950 and link libkap.so; returns its path."""
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
