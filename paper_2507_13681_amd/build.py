"""Builds libloopserve.so (HIP, gfx950) in-tree with hipcc, and _lsnative.so, its Python marshalling, with the C compiler."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_DIR, "csrc")
LIB = os.path.join(_DIR, "libloopserve.so")
NATIVE = os.path.join(_DIR, "_lsnative.so")
SOURCES = ["ls_api.hip", "ls_score.hip", "ls_select.hip", "ls_prefill.hip", "ls_decode.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]


def build_library(verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library; returns its path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for cmd, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + out)
        if verbose and out.strip():
            print(out)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    build_native()
    return LIB


def build_native() -> str:
    """Compile the CPython module that marshals tensors into the C ABI; it finds libloopserve.so beside itself."""
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_path("include"),
           os.path.join(CSRC, "ls_py.c"), "-o", NATIVE, "-L" + _DIR, "-l:libloopserve.so", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("native module failed:\n" + r.stdout)
    return NATIVE


if __name__ == "__main__":
    print(build_library(verbose=True))
