"""Builds libhap.so in-tree with hipcc for gfx950 (no JIT cache: the .so travels with the tree)."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhap.so")
HIP_SOURCES = ["hap_gemm_pp.hip", "hap_gemm_dma.hip", "hap_gemm_small.hip", "hap_gemm_trio.hip", "hap_gemm.hip", "hap_ops.hip", "hap_linear.hip", "hap_moe.hip", "hap_gather.hip", "hap_attn.hip"]
C_SOURCES = ["hap_host.c", "hap_synth.c"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compiles every source and links libhap.so; always recompiles."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    cmds, objs = [], []
    for src in HIP_SOURCES:
        path = os.path.join(CSRC, src)
        if not os.path.exists(path):
            continue
        obj = os.path.join(objdir, src + ".o")
        cmds.append([HIPCC] + HIP_FLAGS + ["-c", path, "-o", obj]); objs.append(obj)
    for src in C_SOURCES:
        obj = os.path.join(objdir, src + ".o")
        cmds.append(["gcc", "-O2", "-Wall", "-Wextra", "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                     "-c", os.path.join(CSRC, src), "-o", obj]); objs.append(obj)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        for out in ex.map(_run, cmds):
            if verbose and out.strip():
                print(out)
    out = _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    if verbose and out.strip():
        print(out)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
