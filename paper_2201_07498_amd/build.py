"""Compiles the gfx950 HIP library liblanczos_topk.so in place."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = [os.path.join(HERE, "csrc", f) for f in ("lz_setup.hip", "lz_step_spmv.hip", "lz_kernels.hip", "lz_finish.hip", "lz_api.hip", "lz_memory.hip", "lz_ooc.hip", "lz_server.hip", "lz_noalloc.hip", "lz_sweep.hip")]
LIB = os.path.join(HERE, "liblanczos_topk.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # Keep the compiler from emitting packed FP32 instructions.
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def build(verbose: bool = False) -> str:
    srcs = [s for s in SRC if os.path.exists(s)]
    tmp = LIB + ".tmp"
    cmd = [HIPCC] + FLAGS + ["-o", tmp] + srcs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
