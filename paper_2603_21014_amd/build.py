"""Builds libclt.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import glob
import os
import re
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libclt.so")
SOURCES = ["clt_api.hip", "kernels_gemm_f32.hip", "kernels_gemm_bf16.hip", "kernels_elementwise.hip", "kernels_gather.hip",
           "kernels_diag.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         # packed fp32 arithmetic is switched off for all device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def vector_work_without_lanes(asm: str) -> list:
    """(kernel, instruction) of every vector instruction that an assembly listing has between the end of a loop over
    lanes and the instruction that gives the wavefront its lanes back.

    A loop that leaves its lanes one by one ends with EXEC empty.  The compiler writes such a loop around every buffer
    access whose descriptor it cannot prove to be the same in all lanes, and its register allocator has put the store
    of a spilled register right behind the loop, in front of the restoring move: nothing is stored, and the reload
    brings whatever the scratch memory held.  (Seen on the row kernel of dW_dec with a descriptor held in vector
    registers and a limit of 72 registers: wrong updates of the weights.)  Reads and writes of single lanes do not look
    at EXEC."""
    found, kernel, empty, last = [], "", False, ""
    for line in asm.splitlines():
        line = line.split(";")[0].strip()
        if not line or line.startswith("."):
            continue
        label = re.match(r"(\S+):$", line)
        if label:
            kernel, empty = label.group(1), False
            continue
        if line.startswith("s_cbranch_execnz"):
            empty = re.match(r"s_\w+ exec,", last) is not None
        elif empty:
            if re.match(r"s_\w+ exec,|s_\w+saveexec|s_branch|s_endpgm", line):
                empty = False
            elif re.match(r"(v_|ds_|buffer_|global_|flat_|scratch_)", line) and not re.match(r"v_(readlane|readfirstlane|writelane)", line):
                found.append((kernel, line))
        last = line
    return found


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    with tempfile.TemporaryDirectory() as tmp:          # -save-temps: the device code's assembly on its way to the object
        cmd = [HIPCC, *FLAGS, "-save-temps", "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True, cwd=tmp)
        listing = glob.glob(os.path.join(tmp, "*gfx950.s"))
        if r.returncode == 0 and len(listing) != 1:
            raise RuntimeError(f"{src}: one listing of the device code expected, found {listing}")
        for f in listing if r.returncode == 0 else ():
            with open(f) as h:
                lost = vector_work_without_lanes(h.read())
            if lost:
                raise RuntimeError(f"{src}: vector instructions with no lane at work, behind a loop over lanes:\n" +
                                   "\n".join(f"  {k}: {i}" for k, i in lost))
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(6, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
