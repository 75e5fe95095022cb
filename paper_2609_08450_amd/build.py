"""Builds the HIP library libtopk_ragged.so in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "csrc", "topk_ragged.hip")
LIB_PATH = os.path.join(HERE, "libtopk_ragged.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc")
                       else (shutil.which("hipcc") or "hipcc"))

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # no packed FP32 instructions anywhere in this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # every atomic here is issued by one lane; the wave-level atomic
    # rewrite only adds instructions and waits for returned values at once
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
    # hoisting out of the machine loops only lengthens live ranges in kernels
    # of this size: without it the instance for planned splits takes 96 vector
    # registers instead of 112, the one for item tables 91 instead of 98, the
    # exact kernel 96 instead of 113 (when it was left out: the decode batch
    # 15.82 us instead of 15.87, the captured decode step 105.4 instead of
    # 106.8, 256 rows 24.1 instead of 24.2, chunked prefill 431.6 instead of
    # 430.6)
    "-mllvm", "-disable-machine-licm",
    "-Wall",
]


def build(verbose: bool = False) -> str:
    cmd = [HIPCC, *FLAGS, "-o", LIB_PATH + ".tmp", SRC]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    msgs = [ln for ln in (res.stdout + res.stderr).splitlines()
            if ln.strip() and "packed-fp32-ops" not in ln]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs))
    os.replace(LIB_PATH + ".tmp", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
