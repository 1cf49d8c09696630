"""Builds libfineserve.so (hipcc, gfx950) next to this file."""
from __future__ import annotations

import os
import shutil
import subprocess
import sysconfig

_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_DIR)
LIB = os.path.join(_DIR, "libfineserve.so")
FAST = os.path.join(_DIR, "_fsfast" + sysconfig.get_config_var("EXT_SUFFIX"))  # (for this interpreter alone)
SOURCES = ["fs_pool.hip", "fs_append.hip", "fs_attention.hip", "fs_attention_generic.hip", "fs_attention_mfma.hip",
           "fs_prefill.hip", "fs_sched.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops off: the compiler must not form packed fp32 instructions.
# -ffp-contract=off: quantizer arithmetic must not be fused (bytes are compared bit for bit).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
FLAGS += os.environ.get("FS_EXTRA_HIPCC_FLAGS", "").split()  # experiments only
# The MFMA kernels keep accumulators and results in vector registers (no AccVGPR operands): their softmax reads every
# S^T tile with the vector ALU, which cannot address AccVGPRs.  (Decode at head_dim 256, the only shape there with more
# than 256 registers: 60 INT8 sequences of 500 - 9000 tokens, 4 KV heads, 146.7 us without the flag, 141.4 with it.)
FILE_FLAGS = {src: ["-mllvm", "-amdgpu-mfma-vgpr-form"] for src in ("fs_prefill.hip", "fs_attention_mfma.hip")}
# Loops begin at half a line of the instruction cache, so that code elsewhere in a kernel does not shift them: a change in what
# runs once, at the launch's end, moved the FP8 prefill loop by 20 bytes and cost it 1.5 - 2 % (24 prompts of 512 - 4096 tokens 1298 ->
# 1323 us; aligned 1298).  Whole lines cost the smallest calls of the 16-column kernel 4 % (one INT8 prompt of 60 tokens at head_dim
# 64 16.9 -> 17.6 us).
FILE_FLAGS["fs_prefill.hip"].append("-falign-loops=32")


TIMELINE_LIB = os.path.join(_DIR, "libfineserve_timeline.so")


def build(verbose: bool = False, timeline: bool = False) -> str:
    """The library; timeline=True: its profiling twin libfineserve_timeline.so (-DFS_TIMELINE: the decode kernel
    leaves clock readings at the end of the workspace; what bench_timeline.py loads, never the product path)."""
    csrc = os.path.join(_DIR, "csrc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(csrc, src.replace(".hip", ".timeline.o" if timeline else ".o"))
        cmd = [HIPCC, *FLAGS, *(["-DFS_TIMELINE"] if timeline else []), *FILE_FLAGS.get(src, []), "-I",
               os.path.join(ROOT, "include"), "-I", csrc, "-c", os.path.join(csrc, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        out = "\n".join(ln for ln in out.splitlines() if "packed-fp32-ops" not in ln)
        if pr.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    if not timeline:  # the binding's native marshaling: a CPython module, no device code; without it calls go through ctypes
        cc = [os.environ.get("CC") or shutil.which("gcc") or os.path.join(os.path.dirname(HIPCC), "amdclang"), "-O2", "-Wall", "-Wextra",
              "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"),
              os.path.join(csrc, "fs_fastcall.c"), "-o", FAST]
        if verbose:
            print(" ".join(cc))
        if os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
            subprocess.run(cc, check=True)
        else:
            print("no Python.h: the binding's small calls go through ctypes (3.5 - 5 us more each)")
    lib = TIMELINE_LIB if timeline else LIB
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-o", lib, *objs], check=True)
    return lib


if __name__ == "__main__":
    import sys

    print(build(verbose=True, timeline="--timeline" in sys.argv[1:]))
