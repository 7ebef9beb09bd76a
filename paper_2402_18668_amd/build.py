"""Builds the HIP library in-tree for gfx950: ``python -m paper_2402_18668_amd.build``."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libbased_hip.so")
BIND = os.path.join(LIBDIR, "_bind.so")

SOURCES = [
    "api.hip",
    "state_io.hip",
    "decode.hip",
    "linattn_prefill_f32.hip",
    "linattn_prefill_f32_dp32.hip",
    "linattn_prefill_f32x3.hip",
    "linattn_prefill_mfma.hip",
    "linattn_prefill_mfma32.hip",
    "linattn_prefill_mfma32_short.hip",
    "swa_prefill_f32.hip",
    "swa_prefill_mfma.hip",
    "swa_prefill_mfma16.hip",
    "linear_mfma.hip",
    "baseconv.hip",
    "rotary.hip",
]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 vector ops are kept out of every device code object
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def bind_command() -> list:
    """The host-only binding module: plain C++ against the Python and torch headers."""
    import sysconfig
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", os.path.join(CSRC, "bind.cpp"), "-o", BIND]
    cmd += ["-I" + d for d in [*include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"]]]
    cmd += ["-L" + d for d in library_paths()]
    return cmd + ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python"]


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every translation unit (in parallel), link the shared library and build the binding module."""
    os.makedirs(LIBDIR, exist_ok=True)
    objdir = os.path.join(LIBDIR, "obj")
    os.makedirs(objdir, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = bind_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs = [("bind.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))]
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed = True
            print(f"[build] {src} FAILED\n{out}", file=sys.stderr)
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("compilation failed")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
