"""Build the HIP library libls.so in-tree for gfx950 with hipcc.

    python -m paper_2510_02483_amd.build      # or build() from Python

Every call recompiles all sources (a few seconds each, in parallel).
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libls.so")
SOURCES = ("abi.hip", "gemm.hip", "gemm_nt.hip", "gemm_nn.hip", "gemm_tn.hip", "attention.hip", "norm.hip", "lmhead.hip", "optim.hip", "headpad.hip")
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-I", INCLUDE, "-I", CSRC,
    # keep the compiler from forming packed fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]

# The attention kernels keep their matrix-product accumulators in ordinary
# vector registers (the softmax works on them), which leaves the accumulation
# registers free for values that only the matrix cores read.
EXTRA = {"attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


def build(verbose: bool = False) -> str:
    """Compile every source and link libls.so next to this file; returns its path."""
    with tempfile.TemporaryDirectory(prefix="ls_build_") as tmp:
        procs = []
        objs = []
        for src in SOURCES:
            obj = os.path.join(tmp, src + ".o")
            objs.append(obj)
            cmd = [HIPCC, *CFLAGS, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        errors = []
        for src, p in procs:
            out, _ = p.communicate()
            text = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip()
                             and "warning generated" not in l)
            if p.returncode != 0:
                errors.append(f"--- {src} ---\n{out}")
            elif verbose and text:
                print(text)
        if errors:
            raise RuntimeError("hipcc failed:\n" + "\n".join(errors))
        tmp_lib = LIB + ".tmp"
        cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp_lib, *objs]
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n" + r.stdout)
        os.replace(tmp_lib, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
