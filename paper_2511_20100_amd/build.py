"""Builds libmtmc.so (HIP, gfx950) in-tree with hipcc.  `python -m paper_2511_20100_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmtmc.so")
SOURCES = ["api.hip", "engine.hip", "engine_bf16.hip", "kernels_f32.hip", "ppo.hip", "probes.hip", "gemm_bf16.hip", "gemm_lds.hip",
           "attention_prefill.hip", "elementwise_bf16.hip", "decode_bf16.hip", "decode_rows128.hip", "decode_lmhead.hip",
           "decode_persistent.hip", "decode_persistent_rows.hip", "decode_persistent_some.hip", "persistent_turn.hip", "rollout_f32.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build()
