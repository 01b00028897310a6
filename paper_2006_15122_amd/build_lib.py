"""Build the HIP library libcosmolat.so for gfx950 (hipcc, in-tree).

Each source is compiled to an object in parallel, its assembly is checked (see
masked_join_writes), then the objects are linked into the shared library next to
this file."""
from __future__ import annotations

import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
SOURCES = ["lattice.hip", "scalar.hip", "fft.hip", "u1.hip", "su2.hip", "noalloc.hip", "batch.hip", "mlp.hip"]
OUT = os.path.join(HERE, "libcosmolat.so")
HIPCC = "/opt/rocm/bin/hipcc"

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # keep the compiler from emitting packed FP32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result", "-Wno-unused-value",
]


def masked_join_writes(asm: str) -> list:
    """Vector instructions that a kernel runs under a branch's lane mask where
    the branch has already been left, as (kernel, label, instructions).

    The block where a divergent branch joins is reached with the branch's mask,
    or with no lane at all where a wave skipped it, and has to widen the mask
    (s_or_b64 exec; s_or_saveexec and s_andn2_saveexec ahead of an else) before
    anything else.  Under register pressure the compiler
    has placed copies of live values, split in two there, ahead of that: the
    other lanes' values were lost.  An FP64 build of the SU(2) x U(1) pass
    computed its second plane from stale LDS addresses that way; nothing in the
    source shows it, and a build whose copies happen to hold rarely used
    constants passes every test."""
    found, kernel, body = [], None, []

    def scan():
        skips = {m.group(1) for m in (re.match(r"s_cbranch_execz (\S+)", s) for s in body) if m}
        block, label, prev = None, "", ""
        for s in body:
            if s.endswith(":"):
                # a join: skipped to, or fallen into past a branch to an out-of-line body
                label = s[:-1]
                block = [] if label in skips or prev.startswith("s_cbranch_execnz") else None
                continue
            prev = s
            if block is None:
                continue
            if s.startswith(("s_or_b64 exec, exec,", "s_or_saveexec_b64", "s_andn2_saveexec_b64")):
                if block:
                    found.append((kernel, label, block))
                block = None
            elif s.startswith(("s_cbranch", "s_branch", "s_barrier", "s_endpgm")) or "exec" in s:
                block = None
            elif s.startswith(("v_", "ds_", "global_", "buffer_", "flat_", "scratch_")) and not s.startswith(
                    ("v_readlane", "v_writelane", "v_readfirstlane")):  # (which take no mask)
                block.append(s)

    for line in asm.splitlines():
        if line.startswith("; %bb."):
            body.append(line.split(":")[0][2:] + ":")  # an unlabelled block
            continue
        s = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):$", s)
        if m or s.startswith(".Lfunc_end"):
            if kernel:
                scan()
            kernel, body = (m.group(1) if m else None), []
        elif kernel and s and (not s.startswith(".") or s.endswith(":")):
            body.append(s)
    return found


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory(prefix="cosmolat_build_") as td:
        procs, objs = [], []
        for s in SOURCES:
            obj = os.path.join(td, s + ".o")
            cmd = [HIPCC, *FLAGS, "-save-temps=obj", "-c", os.path.join(CSRC, s), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((cmd, subprocess.Popen(cmd)))
            objs.append(obj)
        failed = [cmd for cmd, p in procs if p.wait() != 0]
        if failed:
            raise subprocess.CalledProcessError(1, failed[0])
        for s in SOURCES:
            with open(os.path.join(td, os.path.splitext(s)[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")) as f:
                for kernel, label, instrs in masked_join_writes(f.read()):
                    raise RuntimeError(f"{s}: {kernel}: {label} writes registers before the lane mask is restored: "
                                       + "; ".join(instrs))
        tmp = OUT + ".tmp"
        link = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.check_call(link)
        os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
