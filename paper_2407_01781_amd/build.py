"""Compile the HIP sources into paper_2407_01781_amd/libfvdb_hotpath.so (gfx950 only)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfvdb_hotpath.so")
SOURCES = ["conv_wgrad_bf16.hip", "conv_wgrad_f16.hip", "conv.hip", "conv_bwd.hip", "conv_leaf.hip", "conv_lowdepth.hip",
           "grid.hip", "kmap.hip", "conv_wgrad_pairs.hip", "conv_wgrad_lists.hip", "pool.hip", "lib.hip"]      # the ones that take longest first
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _newest_source_mtime() -> float:
    m = 0.0
    for root, _, files in os.walk(CSRC):
        for f in files:
            m = max(m, os.path.getmtime(os.path.join(root, f)))
    m = max(m, os.path.getmtime(os.path.join(os.path.dirname(HERE), "include", "fvdb_hotpath.h")))
    return m


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source to an object (in parallel, one hipcc per file) and link the shared library."""
    if not force and os.path.exists(LIB) and os.path.getmtime(LIB) >= _newest_source_mtime():
        return LIB
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc] + compile_flags + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        return obj, subprocess.run(cmd, capture_output=True, text=True)

    with ThreadPoolExecutor(min(8, len(SOURCES))) as ex:
        results = list(ex.map(compile_one, SOURCES))
    errs = []
    for obj, res in results:
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        if err.strip():
            errs.append(err)
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + [obj for obj, _ in results] + ["-o", LIB]
    if verbose:
        print(" ".join(link))
    res = subprocess.run(link, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose and errs:
        print("\n".join(errs))
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
