"""Builds libsbw.so in-tree with hipcc for gfx950, _binding.so, the Python entry points'
native call path, and libsbw_rate.so, the Philox throughput probe that only the benchmark
loads (neither is part of the ABI)."""
from __future__ import annotations

import importlib.util
import os
import subprocess
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIBRARY = os.path.join(PKG, "libsbw.so")
SOURCES = [os.path.join(CSRC, "sbw_kernels.hip")]
BINDING = os.path.join(PKG, "_binding.so")
BINDING_SOURCE = os.path.join(CSRC, "binding.cpp")
RATE_LIBRARY = os.path.join(PKG, "libsbw_rate.so")
RATE_SOURCES = [os.path.join(CSRC, "philox_rate.hip")]
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
HEADERS = [os.path.join(CSRC, "sbw_device.hpp"), os.path.join(INCLUDE, "sbw.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # bit-exact arithmetic: no FMA contraction, no fast-math, fp32 denormals kept,
    # IEEE-rounded fp32 divide (the sampler's logarithm divides once)
    "-ffp-contract=off",
    "-fno-fast-math",
    "-fno-gpu-flush-denormals-to-zero",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    # packed fp32 VALU ops stay off
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), os.path.join(ROCM, "bin", "hipcc")):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def build(extra_flags: list[str] | None = None, output: str = LIBRARY,
          sources: list[str] | None = None) -> str:
    cmd = [hipcc(), *HIPCC_FLAGS, *(extra_flags or []), "-I", INCLUDE, "-I", CSRC,
           *(sources or SOURCES), "-o", output + ".tmp"]
    subprocess.run(cmd, check=True)
    os.replace(output + ".tmp", output)
    return output


def build_rate() -> str:
    """The benchmark's Philox throughput probe, in a library of its own."""
    return build(output=RATE_LIBRARY, sources=RATE_SOURCES)


def build_binding() -> str:
    """The CPython extension, host code only, against torch's headers and libsbw.so."""
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    lib = os.path.join(torch, "lib")
    include = os.path.join(torch, "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", INCLUDE, "-isystem", include,
           "-isystem", os.path.join(include, "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(ROCM, "include"), "-isystem", sysconfig.get_paths()["include"],
           BINDING_SOURCE, "-o", BINDING + ".tmp", "-L", PKG, "-lsbw", "-L", lib, "-ltorch_python",
           "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + lib]
    subprocess.run(cmd, check=True)
    os.replace(BINDING + ".tmp", BINDING)
    return BINDING


if __name__ == "__main__":
    print(build())
    print(build_binding())
    print(build_rate())
