"""Build libepdlb.so (HIP, gfx950) in-tree with hipcc.

Usage: python -m paper_1804_02883_amd.build   (or build() from Python)
"""
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libepdlb.so")

SOURCES = ["epdlb.hip", "prop_plain.hip"]
HEADERS = ["fft.hpp", "kernels.hpp"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared",
    "--offload-arch=gfx950",
    # no packed-FP32 VALU forms in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # a kernel in a header is inline for the linker's sake; the compiler warns that it cannot be inlined
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable", "-Wno-cuda-compat",
]


PROBES = ("sync_costs", "conv_floor")  # stand-alone programs under probes/ (see their headers)


def build_probe(name, verbose=True):
    src = os.path.join(PKG, "probes", name + ".hip")
    exe = os.path.join(PKG, "probes", name)
    cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", src, "-o", exe + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building the probe " + name)
    os.replace(exe + ".tmp", exe)
    return exe


def build(verbose=True):
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    tmp = LIB + ".tmp"
    cmd = [HIPCC] + FLAGS + ["-I", INCLUDE, "-I", CSRC] + srcs + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed building libepdlb.so")
    # hipcc's host pass warns that it does not know the packed-fp32 feature
    noise = [l for l in (r.stderr or "").splitlines() if l.strip() and "packed-fp32-ops" not in l
             and "not a recognized feature" not in l]
    if verbose and noise:
        sys.stderr.write("\n".join(noise) + "\n")
    os.replace(tmp, LIB)
    for name in PROBES:
        build_probe(name, verbose)
    return LIB


if __name__ == "__main__":
    build()
