"""Build step for the HIP library (gfx950 only).

``python -m paper_2506_05433_amd.build`` (or ``build()``) compiles
``csrc/pg_attn.hip`` with hipcc into ``libpg_attn.so`` next to this file.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "pg_attn.hip")
OUT = os.path.join(HERE, "libpg_attn.so")
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (set HIPCC or install ROCm)")


def command(out: str = OUT, extra=()) -> list:
    return [hipcc(), f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-shared", "-fPIC",
            # packed fp32 VALU forms are kept out of the generated code on purpose
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            # results of matrix products that vector instructions read next stay in VGPRs also in
            # kernels that use AGPRs (pg_bwd_wide.hpp keeps its accumulators there). Of the other
            # kernels it changes the fp32 head_dim 128 forward, dQ and final-token ones (864, 343 and
            # 576 copies between VGPRs and AGPRs become 53, 28 and 32; an fp32 step of 2 x 4, P 257..900,
            # 8/4 heads 601 -> 591 us); the code of the bf16 ones is the same
            "-mllvm", "-amdgpu-mfma-vgpr-form=1",
            "-o", out, SRC, *extra]


def build(verbose: bool = False) -> str:
    tmp = OUT + ".tmp"
    cmd = command(tmp)
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + msgs)
    if verbose and msgs.strip():
        print(msgs)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
