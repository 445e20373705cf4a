"""Builds the HIP library (libmrl.so) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmrl.so")
HOST = os.path.join(HERE, "mrl_host.so")       # the binding's native part (a CPython extension on torch's headers)
SOURCES = ["mrl_api.hip", "mrl_gemm_bf16.hip", "mrl_gemm_f32.hip", "mrl_aux.hip", "mrl_adv.hip", "mrl_probe.hip", "mrl_thl.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build(verbose: bool = True, jobs: int = 4) -> str:
    """Compile every source to an object file, then link the shared library."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        if len(procs) >= jobs:
            _drain(procs)
    _drain(procs)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    _build_host(verbose)
    return LIB


def _build_host(verbose: bool) -> bool:
    """The CPython extension of the binding, linked against libmrl.so beside it.  It needs torch's headers and a host compiler, which
    libmrl.so does not: without them the binding goes through ctypes, and this says so."""
    if os.path.exists(HOST):
        os.remove(HOST)                        # (a stale one must not stay beside a new library)
    try:
        _compile_host(verbose)
        return True
    except (ImportError, OSError, subprocess.CalledProcessError) as e:
        sys.stderr.write(f"warning: {HOST} was not built ({e}); the binding will go through ctypes only\n")
        return False


def _compile_host(verbose: bool):
    import sysconfig

    import torch
    from torch.utils import cpp_extension as ext
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DMRL_TORCH_VERSION="{torch.__version__}"',
           *("-I" + p for p in [*ext.include_paths(), sysconfig.get_paths()["include"]]),
           os.path.join(CSRC, "mrl_host.cpp"), "-o", HOST, *("-L" + p for p in [*ext.library_paths(), HERE]),
           "-lc10", "-ltorch_cpu", "-ltorch_python", "-l:libmrl.so", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)


def _drain(procs):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip()]
        if p.returncode != 0:
            sys.stderr.write("\n".join(lines) + "\n")
            raise RuntimeError(f"hipcc failed on {src}")
        for l in lines:
            if "error" in l or "warning" in l:
                print(l)


if __name__ == "__main__":
    print(build())
