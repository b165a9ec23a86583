"""Builds libmi355gemm.so (HIP, gfx950 only) next to this file with hipcc."""
from __future__ import annotations

import os
import re
import shutil
import subprocess

from .asm_check import Listing, accumulator_hazards, lds_load_hazards

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmi355gemm.so")
SOURCES = [os.path.join(CSRC, f) for f in
           ("gemm_api.hip", "mfma_bf16_inst.hip", "mfma_f16_inst.hip",
            "mfma16_bf16_inst.hip", "mfma16_f16_inst.hip", "mfma16p_bf16_inst.hip", "mfma16p_f16_inst.hip",
            "mfma16t_nn_bf16_inst.hip", "mfma16t_nn_f16_inst.hip", "mfma16t_tn_bf16_inst.hip", "mfma16t_tn_f16_inst.hip",
            "mfma16t_tt_bf16_inst.hip", "mfma16t_tt_f16_inst.hip", "mfma16s_bf16_inst.hip", "mfma16s_f16_inst.hip", "mfma16_f8_inst.hip", "mfma16p_f8_inst.hip", "ring_bf16_inst.hip", "ring_f16_inst.hip", "ring_f8_inst.hip", "mfma16g_inst.hip", "rope_api.hip", "probe_api.hip")]
OBJ_DIR = os.path.join(os.path.dirname(HERE), "_build")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # packed-fp32 VALU forms stay off
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Rpass-analysis=kernel-resource-usage",
         # keep the generated device assembly next to the object: it is scanned below
         "-save-temps=obj"]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the GEMM library cannot be built")


def sources_newer_than_lib() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)]
    deps.append(os.path.join(os.path.dirname(HERE), "include", "gemm.h"))
    deps.append(os.path.join(os.path.dirname(HERE), "include", "rope.h"))
    deps.append(os.path.join(os.path.dirname(HERE), "include", "probe.h"))
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(verbose: bool = False, only: tuple = ()) -> str:
    """Compile every kernel instantiation for gfx950 (one object per translation unit, side by
    side) and link them into one shared library.  `only`: source file names to recompile (the
    other objects are taken as they are; for development, when a change touches one unit)."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(OBJ_DIR, exist_ok=True)
    noise = ("is not a recognized feature for this target", "-Rpass-analysis=kernel-resource-usage")

    def compile_one(src):
        obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
        if only and os.path.basename(src) not in only and os.path.exists(obj):
            return src, obj, subprocess.CompletedProcess([], 0, "", "")
        res = subprocess.run([_hipcc()] + FLAGS + ["-c", src, "-o", obj], capture_output=True, text=True)
        return src, obj, res

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as pool:
        results = list(pool.map(compile_one, SOURCES))
    objs, remarks = [], []
    for src, obj, res in results:
        err = "\n".join(l for l in res.stderr.splitlines() if not any(n in l for n in noise))
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed on {os.path.basename(src)}:\n" + err)
        if verbose and err.strip():
            print(err)
        objs.append(obj)
        remarks.append(res.stderr)
        if res.args and "Function Name:" not in res.stderr:
            raise RuntimeError(f"no resource usage reported for {os.path.basename(src)}: it cannot be checked for scratch memory")
    bad = kernels_with_scratch("\n".join(remarks))
    if bad:
        if os.path.exists(LIB):
            os.remove(LIB)
        raise RuntimeError("kernels that keep data in scratch memory (the hand-scheduled kernels place their own "
                           "waits for asynchronous LDS reads and matrix-core results; a register the compiler "
                           "moves to memory in between breaks that):\n  " + "\n  ".join(bad))
    hazards = []
    for src in SOURCES:
        asm = os.path.join(OBJ_DIR, os.path.splitext(os.path.basename(src))[0] + "-hip-amdgcn-amd-amdhsa-gfx950.s")
        if os.path.exists(asm):
            with open(asm) as f:
                listing = Listing(f.read())
            hazards += [f"{os.path.basename(asm)}:{h}" for h in lds_load_hazards(None, listing) + accumulator_hazards(None, listing)]
    if hazards:
        if os.path.exists(LIB):
            os.remove(LIB)
        raise RuntimeError("a direct-to-LDS load reads a scalar register fewer than 5 wait states after a vector-ALU "
                           "instruction wrote it, an MFMA a register fewer than 2 after one wrote it, or another instruction an "
                           "accumulator fewer than 19 after an MFMA wrote it:\n  " + "\n  ".join(hazards[:20]))
    res = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC",
                          "-Wl,--version-script=" + os.path.join(CSRC, "exports.map"), "-o", LIB] + objs,
                         capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("linking failed:\n" + res.stderr)
    return LIB


def kernels_with_scratch(remarks: str) -> list:
    """Names of kernels whose resource-usage remarks show scratch memory or vector-register spills
    (scalar registers spilled into vector-register lanes stay in registers and are fine).  The compiler writes
    "file:line: remark: text", and with -save-temps, where it compiles in steps, "remark: file:line: text"."""
    bad, name = [], None
    for what, value in re.findall(r"remark:.*?\b(Function Name|ScratchSize \[bytes/lane\]|VGPRs Spill): *([^\s\[]+)", remarks):
        if what == "Function Name":
            name = value
        elif int(value) != 0 and name not in bad:
            bad.append(name)
    return bad


if __name__ == "__main__":
    print(build_library(verbose=True))
