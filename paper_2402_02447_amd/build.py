"""Compile libbca.so (host side + HIP kernels of the clip + optimizer path, and the load-balancing
simulation) for gfx950, and the extension module _calls that Python makes its compute calls through, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbca.so")
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
SOURCES = [os.path.join(CSRC, "bca_host.cpp"), os.path.join(CSRC, "bca_kernels.hip"), os.path.join(CSRC, "lbs.hip")]

# Packed fp32 instructions are switched off for all device code.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-command-line-argument", "-x", "hip",
]


def build(verbose: bool = False, extra: list | None = None, out: str = LIB) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *HIPCC_FLAGS, *(extra or []), "-I", os.path.join(ROOT, "include"), "-I", CSRC, *SOURCES, "-o", out]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    if out == LIB:  # the package as it is imported: both parts
        build_calls()
    return out


def build_calls(out: str = CALLS) -> str:
    """The extension module: host code that includes bca.h and links nothing."""
    subprocess.run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra", "-Wno-missing-field-initializers",
                    "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "calls.cpp"), "-o", out], check=True)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
