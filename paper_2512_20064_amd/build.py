"""Build libmps.so (the C-ABI library with its gfx950 HIP kernels) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmps.so")
ARCH = "gfx950"

SOURCES = ["mps_abi.cpp", "contract_f32.hip", "contract_lp.hip", "measure.hip", "decompress.hip", "sweep_small.hip", "sweep_mid.hip",
           "sweep_mid_f32.hip"]

# -packed-fp32-ops off: no v_pk_{add,mul,fma}_f32 in the device code.
HIP_FLAGS = ["-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-result"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link libmps.so; returns its path."""
    objs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"]
        cmd = [hipcc(), *HIP_FLAGS, *lang, "-I", os.path.join(ROOT, "include"), "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


def build_checks(verbose: bool = False) -> str:
    """Compile the device checks of the tests (tests/e2m3_device.hip) to
    tests/libe2m3_device.so; returns its path."""
    tests = os.path.join(ROOT, "tests")
    lib = os.path.join(tests, "libe2m3_device.so")
    cmd = [hipcc(), *HIP_FLAGS, "-x", "hip", "-I", CSRC, "-shared", os.path.join(tests, "e2m3_device.hip"),
           "-o", lib + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(lib + ".tmp", lib)
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
