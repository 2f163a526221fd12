"""Builds the HIP library in-tree: hipcc cross-compiles for gfx950 without a GPU."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libstripe_hip.so")
SOURCES = ["api.cpp", "plan.cpp", "tiling.cpp", "generic.hip", "generic_tiled.hip", "contract.hip:4", "contract.hip:2", "contract.hip:1", "pool.hip", "gemm.hip", "gemm_rows.hip", "conv.hip", "conv_i8.hip", "conv_igemm.hip", "conv_few.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
         # the LDS-direct load helpers name M0 in their clobber lists on purpose (see their comments); the compiler
         # notes that it treats M0 as reserved, once per unrolled copy
         "-Wno-inline-asm"]


def needs_build() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(HERE, "..", "include", "stripe.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not needs_build():
        return LIB
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        # "file:n": the file compiled with CONTRACT_T = n (element size of the kernels in that object)
        src, _, elem = src.partition(":")
        obj = os.path.join(HERE, "_build", src + elem + ".o")
        cmd = ["hipcc"] + [f for f in FLAGS if f != "-shared"] + ([f"-DCONTRACT_T={elem}"] if elem else []) + ["-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        objs.append(obj)
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        text = "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            print(f"--- {src} failed\n{text}", file=sys.stderr)
        elif verbose and text.strip():
            print(f"--- {src}\n{text}")
    if failed:
        raise RuntimeError("hipcc failed")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
