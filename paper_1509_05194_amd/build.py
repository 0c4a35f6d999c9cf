"""Builds libhclae.so (HIP, gfx950 only) in-tree next to this file."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhclae.so")
PROBE = os.path.join(HERE, "libhclae_probe.so")      # for the tests: single instructions of the contraction

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-shared", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return [os.path.join(CSRC, "hclae.hip")]


def build(verbose=False, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc] + HIPCC_FLAGS + list(extra) + ["-o", LIB] + sources()
    for c in (cmd, [hipcc] + HIPCC_FLAGS + list(extra) + ["-o", PROBE, os.path.join(CSRC, "probe.hip")]):
        if verbose:
            print(" ".join(c))
        subprocess.run(c, check=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    print(LIB)
