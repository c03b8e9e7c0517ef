"""Compile libdn (HIP, gfx950 only) into paper_2001_04206_amd/libdn.so.

Every source is compiled to an object of its own (in parallel, into _build/), then linked.
"""
from __future__ import annotations

import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdn.so")
SOURCES = ["dn_api.hip", "dn_gemm.hip", "dn_small.hip", "dn_online.hip", "dn_twin.hip", "dn_solo.hip", "dn_tiny.hip", "dn_wide.hip", "dn_block.hip", "dn_block_tanh.hip", "dn_block_relu.hip", "dn_wide_block.hip", "dn_tiles.hip", "dn_slices.hip", "dn_conv.hip", "dn_cnn.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]
HIPCC = "/opt/rocm/bin/hipcc"
# Kernels whose LDS reads are written in assembler must keep their values in registers: a build in which one of them
# spilled has given a wrong sum, for a reason that is not known.  The build fails if one uses scratch memory.
REGISTERS_ONLY = ("SliceTile", "corr3_split_kernel")
REMARKS = "-Rpass-analysis=kernel-resource-usage"


def kernels_with_scratch(remarks: str):
    """Names (mangled) of REGISTERS_ONLY kernels that the compiler's remarks give scratch memory; and how many they name."""
    name, spilled, seen = "", [], 0
    for line in remarks.splitlines():
        m = re.search(r"remark: .*?(Function Name|ScratchSize \[bytes/lane\]): (\S+)", line)
        if not m:
            continue
        if m.group(1) == "Function Name":
            name = m.group(2)
        elif any(k in name for k in REGISTERS_ONLY):
            seen += 1
            if int(m.group(2)):
                spilled.append("%s (%s bytes)" % (name, m.group(2)))
    return spilled, seen


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    text = res.stdout + res.stderr
    out = "\n".join(l for l in text.splitlines()
                    if "is not a recognized feature for this target" not in l and "[-Rpass-analysis" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if REMARKS in cmd:
        spilled, seen = kernels_with_scratch(text)
        if spilled or not seen:
            obj = cmd[-1]
            if os.path.exists(obj):
                os.remove(obj)
            raise RuntimeError("scratch memory in kernels that must not use it: %s" % (spilled or "none of them named"))
    if verbose and out.strip():
        print(out)


def build(verbose: bool = False, only_stale: bool = False) -> str:
    """Compile and link.  only_stale: reuse objects newer than their source and every header."""
    os.makedirs(OBJ, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers.append(os.path.join(HERE, "..", "include", "dn.h"))
    newest_header = max(os.path.getmtime(h) for h in headers)
    jobs = []
    objs = []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src) + ".o")
        objs.append(obj)
        if only_stale and os.path.exists(obj) and os.path.getmtime(obj) >= max(os.path.getmtime(src), newest_header):
            continue
        check = [REMARKS] if os.path.basename(src) in ("dn_gemm.hip", "dn_conv.hip") else []
        jobs.append([HIPCC, *FLAGS, *check, "-I", os.path.join(HERE, "..", "include"), "-c", src, "-o", obj])
    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as pool:
        list(pool.map(lambda c: _run(c, verbose), jobs))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, only_stale="--stale" in sys.argv))
    sys.exit(0)
