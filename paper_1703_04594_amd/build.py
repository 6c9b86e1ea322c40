"""Build step of the GPU library: compiles liblbm.so for gfx950 in-tree.

The constants header is generated by ``csrc/gen_d2q37_tables.py``; the build
checks that the committed header matches the generator's output.
"""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "liblbm.so")
# reference copy kernel used by the benchmark for roofline calibration
PROBE_LIB = os.path.join(HERE, "libcopyprobe.so")
SOURCES = ["lbm_api.hip"]
HEADERS = ["lbm_site.hpp", "lbm_kernels.hpp", "lbm_twostep.hpp", "lbm_adjoint.hpp", "lbm_adjoint_api.inc", "lbm_layouts.hpp", "lbm_layouts_api.inc", "lbm_rollout.h",
           "lbm_hetero_api.inc", "host_band.h", "d2q37_tables.h"]
# host-core part of co-execution: plain C++ with OpenMP, built by the host
# compiler (AVX2 + FMA, so it runs on any x86-64-v3 host) and linked in
HOST_SOURCES = ["host_band.cpp"]
CXX_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-march=x86-64-v3", "-ffp-contract=fast", "-fopenmp"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # no packed FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def check_tables() -> None:
    gen = os.path.join(CSRC, "gen_d2q37_tables.py")
    with tempfile.TemporaryDirectory() as td:
        out = os.path.join(td, "t.h")
        subprocess.run([sys.executable, gen, out], check=True, stdout=subprocess.DEVNULL)
        with open(out) as a, open(os.path.join(CSRC, "d2q37_tables.h")) as b:
            if a.read() != b.read():
                raise RuntimeError("csrc/d2q37_tables.h is out of date: run csrc/gen_d2q37_tables.py")


def build_library(verbose: bool = False) -> str:
    check_tables()
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cxx = os.environ.get("CXX", "g++")
    objs = []
    with tempfile.TemporaryDirectory() as td:
        for src in HOST_SOURCES:
            obj = os.path.join(td, os.path.splitext(src)[0] + ".o")
            cmd = [cxx, *CXX_FLAGS, f"-I{CSRC}", "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd))
            r = subprocess.run(cmd, capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError("host compiler failed:\n" + r.stdout + r.stderr)
            objs.append(obj)
        cmd = [hipcc, *HIPCC_FLAGS, f"-I{INCLUDE}", f"-I{CSRC}",
               *[os.path.join(CSRC, s) for s in SOURCES], "-x", "none", *objs, "-lgomp", "-o", LIB + ".tmp"]
        if verbose:
            print(" ".join(cmd))
        r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout + r.stderr)
    os.replace(LIB + ".tmp", LIB)
    cmd = [hipcc, *HIPCC_FLAGS, f"-I{CSRC}", os.path.join(CSRC, "copy_probe.hip"), "-o", PROBE_LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout + r.stderr)
    os.replace(PROBE_LIB + ".tmp", PROBE_LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
