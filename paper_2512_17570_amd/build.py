"""hipcc build of libgs.so for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libgs.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared",
    "-ffp-contract=off",                     # one rounding per operation: partition-independent results
    "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU forms
    "-mllvm", "-amdgpu-kernarg-preload-count=14",   # leading arguments in registers as a wave starts, up to all there is room for
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build(verbose: bool = True, extra_flags=(), out: str | None = None) -> str:
    out = out or LIB
    cmd = [HIPCC, *FLAGS, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *sources(), "-o", out]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass warns that it does not know the packed-fp32 feature: harmless, filter it
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("hipcc failed")
    if verbose and err.strip():
        print(err)
    return out


PROBE_LIB = os.path.join(PKG, "libgs_mixprobe.so")


def build_probe(verbose: bool = True) -> str:
    """The stream-mix probe bench.py times next to the step kernel (probe/gs_mixprobe.hip): its own
    shared library, so that libgs.so holds the product path only."""
    cmd = [HIPCC, *FLAGS, os.path.join(PKG, "probe", "gs_mixprobe.hip"), "-o", PROBE_LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("hipcc failed (mix probe)")
    return PROBE_LIB


CALL_MODULE = os.path.join(PKG, "_gs_call.so")


def build_call(verbose: bool = True) -> str:
    """The binding's native marshalling (csrc/gs_call.cpp): a CPython extension over torch's headers."""
    import sysconfig

    from torch.utils import cpp_extension
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include"),
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
           "-isystem", sysconfig.get_paths()["include"], *[x for d in cpp_extension.include_paths() for x in ("-isystem", d)],
           os.path.join(CSRC, "gs_call.cpp"), "-o", CALL_MODULE, *[f"-L{d}" for d in cpp_extension.library_paths()],
           "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stderr)
        raise RuntimeError("g++ failed (gs_call)")
    return CALL_MODULE


if __name__ == "__main__":
    build()
    build_probe()
    build_call()
