"""Build libstill.so (HIP, gfx950) in-tree with hipcc.

The library is five translation units compiled in parallel (the C ABI and
the consumer attention; the fp16 attention kernels; the per-layer launch sequence for bf16 I/O; the same
for the fp32 validation mode; the backward pass) and linked into one shared
object."""
from __future__ import annotations

import os
import re
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libstill.so")
CSRC = os.path.join(PKG, "csrc")
SOURCES = [os.path.join(CSRC, f) for f in ("still.hip", "xattn.hip", "layer_bf16.hip", "layer_fp32.hip",
                                            "backward.hip")]
HEADERS = [os.path.join(CSRC, f) for f in ("common.hpp", "gemm.hpp", "attn.hpp", "misc.hpp", "kproj.hpp",
                                           "consumer.hpp", "refine.hpp", "refine64.hpp", "host.hpp",
                                           "layer.hpp", "bwd.hpp")] + [os.path.join(ROOT, "include", "still.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         # keep hipcc from forming packed fp32 (v_pk_*_f32) instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # MFMA operands/results in VGPRs; AGPRs then serve as fast spill space
         "-mllvm", "-amdgpu-mfma-vgpr-form=1"]


def _filter(stderr: str) -> str:
    return "\n".join(l for l in stderr.splitlines() if "packed-fp32-ops" not in l)


def accumulation_register_uses(asm: str) -> list:
    """Uses of an accumulation register by the fp16 attention kernels outside
    inline assembly, which names those that hold their accumulators outright: a
    value of the compiler's there would overwrite them, or be overwritten."""
    inside, kernel, found = False, "", []
    for line in asm.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            kernel = m.group(1)
        if "#ASMSTART" in line:
            inside = True
        elif "#ASMEND" in line:
            inside = False
        elif not inside and line.startswith("\t") and not line.startswith(("\t.", "\t;")):
            if re.search(r"accvgpr|\ba\[?\d", line.split(";")[0]) and "xattn_f16" in kernel:
                found.append(f"{kernel}: {line.strip()}")
    return found


def scratch_bytes(asm: str) -> dict:
    """Scratch bytes per lane of each fp16 attention kernel."""
    sizes = {}
    for m in re.finditer(r"^\s+\.name:\s+(_Z\w+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", asm, re.M):
        if "xattn_f16" in m.group(1):
            sizes[m.group(1)] = int(m.group(2))
    return sizes


def build_library(verbose: bool = False) -> str:
    """Compile the HIP library; always recompiles. Returns the library path."""
    objs = [os.path.join(CSRC, os.path.basename(src) + ".o") for src in SOURCES]
    procs = []
    for src, obj in zip(SOURCES, objs):
        cmd = [HIPCC, *FLAGS, "-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append(subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True))
    asm = os.path.join(CSRC, "xattn.s.o")
    procs.append(subprocess.Popen([HIPCC, *FLAGS, "--cuda-device-only", "-S", "-o", asm, SOURCES[1]],
                                  stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True))
    errors = []
    for src, p in zip([*SOURCES, SOURCES[1]], procs):
        out, err = p.communicate()
        err = _filter(err)
        if p.returncode != 0:
            errors.append(f"{os.path.basename(src)}: hipcc failed ({p.returncode}):\n{err}")
        elif verbose and err.strip():
            print(err, file=sys.stderr)
    if errors:
        raise RuntimeError("\n".join(errors))
    with open(asm) as f:
        found = accumulation_register_uses(f.read())
    os.remove(asm)
    if found:
        raise RuntimeError("this compiler uses accumulation registers that the fp16 attention kernels name:\n"
                           + "\n".join(found[:5]))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed ({r.returncode}):\n{_filter(r.stderr)}")
    os.replace(tmp, LIB)
    for obj in objs:
        os.remove(obj)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
