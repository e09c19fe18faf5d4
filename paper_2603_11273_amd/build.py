"""Builds the HIP library libasr_mi355x.so in-tree for gfx950 (MI355X), and
the seeded input generator libasr_synth.so (test and benchmark input only).

    python -m paper_2603_11273_amd.build

Every HIP source is compiled with hipcc for gfx950 only; the host-only queue
with g++.  Objects go to _build/ next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libasr_mi355x.so")
SYNTH_LIB = os.path.join(HERE, "libasr_synth.so")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")

HIP_SOURCES = ["k_misc.hip", "k_gemm.hip", "k_attn.hip", "k_rows.hip", "runtime.hip"]
CPP_SOURCES = ["queue.cpp", "serve.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed fp32 instructions are disabled: hipcc emits them from plain float
# code at -O3 and we keep all fp32 arithmetic scalar.
# code object v5: loadable by the HIP runtime torch ships as well as by /opt/rocm's.
HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-mcode-object-version=5",
             "-I", INCLUDE,
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-result"]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("build failed:\n" + " ".join(cmd) + "\n" + r.stdout)
    return r.stdout


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    jobs = []
    for src in HIP_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        jobs.append([HIPCC, *HIP_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj])
    jobs.append([HIPCC, *HIP_FLAGS, "-c", os.path.join(CSRC, "synth_gen.hip"), "-o",
                 os.path.join(BUILD, "synth_gen.hip.o")])
    for src in CPP_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        jobs.append(["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-c",
                     os.path.join(CSRC, src), "-o", obj])
    workers = min(len(jobs), max(1, min(8, os.cpu_count() or 1)))
    with ThreadPoolExecutor(workers) as ex:
        outs = list(ex.map(_run, jobs))
    if verbose:
        for o in outs:
            if o.strip():
                print(o)
    objs = [os.path.join(BUILD, s + ".o") for s in HIP_SOURCES + CPP_SOURCES]
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "--offload-arch=gfx950", "-mcode-object-version=5", "-fPIC", "-o",
          tmp, *objs])
    os.replace(tmp, LIB)
    tmp = SYNTH_LIB + ".tmp"
    _run([HIPCC, "-shared", "--offload-arch=gfx950", "-mcode-object-version=5", "-fPIC", "-o",
          tmp, os.path.join(BUILD, "synth_gen.hip.o")])
    os.replace(tmp, SYNTH_LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
