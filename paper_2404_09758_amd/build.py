"""Build libdr.so in-tree with hipcc for gfx950.

Flags: -ffp-contract=off keeps every fp32 expression the correctly rounded
result of its written operation sequence (no fused multiply-add), which the
bit-exact reproducibility of the estimator relies on; packed fp32 ops are
disabled.
"""
from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = [os.path.join(CSRC, f) for f in (
    "dr_kernels.hip", "dr_tile8.hip", "dr_tile16.hip", "dr_tile32.hip", "dr_tile8_deep.hip", "dr_tile16_deep.hip",
    "dr_api.hip", "dr_subdiv.cpp", "dr_probe.hip")]
OUT = os.path.join(HERE, "libdr.so")

HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-fPIC",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def build_lib(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = OUT + ".tmp"
    with tempfile.TemporaryDirectory() as work:
        # one compiler run per source, side by side
        objs = [os.path.join(work, os.path.basename(src) + ".o") for src in SOURCES]
        cmds = [[hipcc] + HIPCC_FLAGS + ["-c", "-o", obj, src] for src, obj in zip(SOURCES, objs)]
        if verbose:
            for cmd in cmds:
                print(" ".join(cmd), flush=True)
        procs = [subprocess.Popen(cmd) for cmd in cmds]
        codes = [p.wait() for p in procs]
        for cmd, code in zip(cmds, codes):
            if code:
                raise subprocess.CalledProcessError(code, cmd)
        subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-o", tmp] + objs)
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build_lib(verbose=True))
