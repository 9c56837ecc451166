"""Build liblbm_hip.so (gfx950) in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbm_hip.so")
SOURCES = ["lbm_kernels.hip", "lbm_march.hip", "lbm_stack.hip", "lbm_api.hip", "lbm_batch.hip"]
ARCH = "gfx950"

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed FP32 instructions stay off: their use is left to nobody
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # contraction only inside one expression: every kernel instance that
    # inlines the node update rounds it identically
    "-ffp-contract=on",
    "-Wall", "-Wno-unused-result",
]


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compile the sources side by side and link them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        jobs, objects = [], []
        for src in SOURCES:
            objects.append(os.path.join(tmp, src + ".o"))
            cmd = [hipcc] + FLAGS + (extra or []) + ["-c", os.path.join(CSRC, src), "-o", objects[-1]]
            if verbose:
                print(" ".join(cmd), flush=True)
            jobs.append((cmd, subprocess.Popen(cmd)))
        codes = [p.wait() for _, p in jobs]
        for (cmd, _), rc in zip(jobs, codes):
            if rc:
                raise subprocess.CalledProcessError(rc, cmd)
        subprocess.run([hipcc, "-shared", f"--offload-arch={ARCH}"] + objects + ["-o", LIB + ".tmp"],
                       check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
