"""Builds the HIP shared library for gfx950 in-tree with hipcc."""

from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB_NAME = "libpalu_hip.so"
LIB_PATH = os.path.join(HERE, LIB_NAME)

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",     # no packed-FP32 VALU forms
    "-fno-fast-math", "-ffp-contract=off",
    "-Wall", "-Wno-unused-function",
]
# The matrix instructions of the attention kernels write ordinary vector registers, so their float32
# epilogues read the accumulators without a copy per value; the prompt-sized projection keeps its 256
# accumulators per lane in the accumulation registers and is compiled on its own without the option.
# (The shared-key forms of the whole-head score kernel unroll 64 matrix instructions with the vector work of up to
# eight queries dealt out between them: beyond the default size limit of "#pragma unroll".)
VGPR_FORM = ["-mllvm", "-amdgpu-mfma-vgpr-form", "-mllvm", "-pragma-unroll-threshold=200000"]
BUILD_DIR = os.path.join(HERE, "_build")


FLAT = ["-DPALU_SCORE_FLAT=1"]


def sources():
    """(source file, extra flags, object name) of every translation unit."""
    vgpr = ["score16_shared_forms.hip", "score_forms.hip", "score_forms_lowbit.hip", "score16_forms.hip", "pv.hip", "api.hip"]
    units = [(f, VGPR_FORM, "") for f in vgpr]
    units += [(f, VGPR_FORM + FLAT, "_flat") for f in ("score16_shared_forms.hip", "score16_forms.hip")]
    units += [("attend16_forms.hip", VGPR_FORM, ""), ("attend16_forms.hip", VGPR_FORM + FLAT, "_flat"), ("attend16_forms.hip", VGPR_FORM + ["-DPALU_ATTEND_SHARED=1"], "_shared"),
              ("attend16_forms.hip", VGPR_FORM + ["-DPALU_ATTEND_SHARED=2"], "_shared_few")]
    units += [("attend16_mixed_forms.hip", VGPR_FORM, "")]
    units += [("encode_gemm.hip", [], "")]
    return [(os.path.join(CSRC, f), extra, os.path.splitext(f)[0] + suffix + ".o") for f, extra, suffix in units]


def _run(procs, verbose):
    for cmd, proc in procs:
        out = proc.communicate()[0]
        lines = [l for l in out.splitlines() if "packed-fp32-ops' is not a recognized feature" not in l]
        if verbose and lines:
            print("\n".join(lines), flush=True)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + "\n".join(lines))


def build_library(verbose: bool = True) -> str:
    """Compile csrc/ into libpalu_hip.so next to this file and return its path."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    os.makedirs(BUILD_DIR, exist_ok=True)
    inc = ["-I", os.path.join(HERE, "..", "include")]
    objects, procs = [], []
    for src, extra, name in sources():
        obj = os.path.join(BUILD_DIR, name)
        cmd = [hipcc] + HIPCC_FLAGS + extra + inc + ["-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objects.append(obj)
    _run(procs, verbose)
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH] + objects
    if verbose:
        print(" ".join(link), flush=True)
    _run([(link, subprocess.Popen(link, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))], verbose)
    return LIB_PATH


if __name__ == "__main__":
    build_library()
    sys.exit(0)
