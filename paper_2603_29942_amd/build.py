"""Build the HIP library ``libbz.so`` for gfx950, in-tree.

    python -m paper_2603_29942_amd.build

One translation unit (``csrc/bz_api.hip``) holds the C ABI of ``include/bz.h``
and instantiates every kernel.  Packed-FP32 instruction selection is switched
off for all device code.

The build fails if an enumeration kernel spills vector registers: the compiler
(ROCm 7.2) has placed the spill of a value that lives through a divergent
region before the region's end restores the execution mask, so that the lanes
outside the region lost it (counts and minima were wrong).
"""
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "csrc", "bz_api.hip")
LIB = os.path.join(HERE, "libbz.so")
ARCH = "gfx950"


def vgpr_spills(remarks: str) -> dict:
    """Kernel name -> spilled vector registers, from the compiler's resource remarks."""
    out, name = {}, None
    for line in remarks.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"VGPRs Spill: (\d+)", line)
        if m and name:
            out[name] = int(m.group(1))
    return out


def build(verbose: bool = False, extra=()) -> str:
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-function", "-Rpass-analysis=kernel-resource-usage",
           "-I", os.path.join(ROOT, "include"), SRC, "-o", LIB + ".tmp", *extra]
    if verbose:
        print(" ".join(cmd), flush=True)
    run = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
    if run.returncode != 0:
        sys.stderr.write(run.stderr)
        raise subprocess.CalledProcessError(run.returncode, cmd)
    spills = vgpr_spills(run.stderr)
    enum = {k: v for k, v in spills.items() if "enum" in k}
    bad = {k: v for k, v in enum.items() if v}
    if not enum or bad:
        raise RuntimeError(f"enumeration kernels must not spill vector registers: {bad or 'no kernel was reported'}")
    for line in run.stderr.splitlines():  # what is left of the compiler's messages
        if re.search(r"(warning|error):", line) and "packed-fp32-ops" not in line:
            print(line, file=sys.stderr)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
