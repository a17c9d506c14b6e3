"""Builds libminions_verify.so (HIP, gfx950) in-tree with hipcc.  No torch involvement."""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libminions_verify.so")
SOURCES = ("api.hip", "vote_accept.hip", "rows.hip", "gemm.hip", "gemm_small.hip", "attention.hip", "stochastic.hip", "probe.hip", "selector.cpp")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-variable",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16"]  # leading kernel arguments in scalar registers (csrc/launch.h)


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library; always recompiles."""
    hipcc = _hipcc()
    extra = os.environ.get("MN_EXTRA_HIPCC_FLAGS", "").split()
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    jobs = []
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        for src in SOURCES:
            obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
            objs.append(obj)
            jobs.append(ex.submit(_run, [hipcc, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]))
        for src, j in zip(SOURCES, jobs):
            out = j.result()
            if verbose and out.strip():
                print("[%s]\n%s" % (src, out))
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
