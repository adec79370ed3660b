"""Builds librlhf_rollout.so for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librlhf_rollout.so")
SOURCES = ["api.hip", "gemm.hip", "gemm_skinny.hip", "few_rows.hip", "decode.hip", "attention.hip", "elementwise.hip", "ppo_signals.hip", "optimizer.hip", "head_backward.hip", "attention_backward.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wno-unused-result",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False) -> str:
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
        if verbose:
            sys.stderr.write(r.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    # stand-alone kernel drivers (hardware-counter runs): each links the library's own object
    for drv, obj in (("gemm_driver", "gemm.o gemm_skinny.o few_rows.o"), ("attn_driver", "attention.o"),
                     ("dec_driver", "gemm.o gemm_skinny.o few_rows.o"), ("ceilings_driver", "")):
        drv_obj = os.path.join(objdir, drv + ".o")
        r = subprocess.run([hipcc, *FLAGS, "-c", os.path.join(CSRC, drv + ".hip"), "-o", drv_obj],
                           capture_output=True, text=True)
        if r.returncode == 0:
            r = subprocess.run([hipcc, "--offload-arch=gfx950", "-o", os.path.join(HERE, drv), drv_obj,
                                *[os.path.join(objdir, o) for o in obj.split()]], capture_output=True, text=True)
        if r.returncode != 0:  # the drivers are measurement aids: the library itself is built, so only warn
            sys.stderr.write(f"warning: {drv} was not built:\n{r.stderr}\n")
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
