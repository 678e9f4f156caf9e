"""Build the HIP library libphx.so for gfx950 (in-tree), and the benchmark's probe library."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libphx.so")
SOURCES = ["phx_api.cpp", "phx_trace.hip", "phx_readout.hip", "phx_moments.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -disable-machine-licm: the kernels loop over photons, and the pass moves the 64-bit constants of exp,
# log, sine and the polynomials out of the loop into vector registers that the whole body
# then holds: 123 instead of 61 registers in the sky kernel, 168 and spills instead of 119 in the optics
# kernel (1e9 photons 40.2 ms with the pass, 37.4 without)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-disable-machine-licm",
         "-Wall", "-Wno-unused-function"]


# the benchmark's memory-system probe, a library of its own (not part of the trace)
PROBE_LIB = os.path.join(HERE, "libphx_probe.so")
PROBE_SOURCES = ["probe.hip"]


def _link(lib, sources, verbose):
    srcs = [os.path.join(CSRC, s) for s in sources]
    tmp = lib + ".tmp"
    cmd = [HIPCC, *FLAGS, "-o", tmp, *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    _link(LIB, SOURCES, verbose)
    _link(PROBE_LIB, PROBE_SOURCES, verbose)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
