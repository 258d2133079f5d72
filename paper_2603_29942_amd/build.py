"""Build the HIP library ``libbz.so`` for gfx950, in-tree.

    python -m paper_2603_29942_amd.build

One translation unit (``csrc/bz_api.hip``) holds the C ABI of ``include/bz.h``
and instantiates every kernel.  Packed-FP32 instruction selection is switched
off for all device code.

The build fails if a kernel spills vector registers: the compiler (ROCm 7.2)
has placed the spill of a value that lives through a divergent region before
the region's end restores the execution mask, so that the lanes outside the
region lost it (counts and minima were wrong).  The compiler's remarks tell the
spills of kernels only, so every device function has to be inlined as well, and
the listing must hold no call and no access to scratch memory.
"""
import os
import re
import shutil
import subprocess
import sys
import tempfile

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


def outside_registers(listing: str) -> dict:
    """Function name -> its calls and accesses to scratch memory, from the device code's listing."""
    out, name = {}, None
    for line in listing.splitlines():
        m = re.match(r"([A-Za-z_.$][\w.$]*):\s*; @", line)
        if m:
            name = m.group(1)
        elif name and re.search(r"^\s*(s_swappc_b64|s_call_b64|scratch_|buffer_(load|store)\w*.*\boffen\b)|; .*Folded ", line):
            out.setdefault(name, []).append(line.strip())
    return out


def check(remarks: str, listing: str) -> None:
    """Raises RuntimeError for spilled vector registers, calls and scratch accesses."""
    spills = vgpr_spills(remarks)
    bad = {k: v for k, v in spills.items() if v}
    if not spills or bad:
        raise RuntimeError(f"kernels must not spill vector registers: {bad or 'no kernel was reported'}")
    outside = outside_registers(listing)
    if outside or "; @" not in listing:
        raise RuntimeError(f"device code must not call or use scratch memory: {outside or 'no listing'}")


def build(verbose: bool = False, extra=()) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        cmd = ["hipcc", f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
               "-Wall", "-Wno-unused-function", "-Rpass-analysis=kernel-resource-usage", "-save-temps=obj",
               "-I", os.path.join(ROOT, "include"), SRC, "-o", os.path.join(tmp, "libbz.so"), *extra]
        if verbose:
            print(" ".join(cmd), flush=True)
        run = subprocess.run(cmd, stderr=subprocess.PIPE, text=True)
        if run.returncode != 0:
            sys.stderr.write(run.stderr)
            raise subprocess.CalledProcessError(run.returncode, cmd)
        listings = [f for f in os.listdir(tmp) if f.endswith(".s") and ARCH in f]
        check(run.stderr, "".join(open(os.path.join(tmp, f)).read() for f in listings))
        for line in run.stderr.splitlines():  # what is left of the compiler's messages
            if re.search(r"(warning|error):", line) and "packed-fp32-ops" not in line:
                print(line, file=sys.stderr)
        shutil.copy(os.path.join(tmp, "libbz.so"), LIB + ".tmp")
        os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
