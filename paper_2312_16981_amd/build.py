"""Compile the HIP sources into paper_2312_16981_amd/libugkwp.so for gfx950.

Floating-point contraction is off in all device code: the particle push and
the sampling take discrete decisions (collision tests, face crossings,
particle counts) whose rounding must be exactly that of the written
expressions.  Packed-FP32 instruction selection is disabled.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libugkwp.so")
SOURCES = ["kernels.hip", "si_tile.hip", "si_grid.hip", "adjoint.hip", "runtime.hip"]
# The tile sweeps loop over code full of 64-bit constants (exp, the Planck
# polynomials); hoisted out of the loop they fill the register file (256 VGPRs and
# spills; as it is 48 to 239 VGPRs, 8 bytes of scratch in two forms), so they are
# formed where they are used.
EXTRA = {"si_tile.hip": ["-mllvm", "-disable-machine-licm"]}
ARCH = os.environ.get("UGKWP_OFFLOAD_ARCH", "gfx950")


def hipcc():
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.isabs(c) and os.path.exists(c):
            return c
    return "hipcc"


def build(verbose=False, jobs=2):
    flags = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-function", "-Wno-unused-result"]
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc(), *flags, *EXTRA.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    for p, cmd in procs:
        if p.wait() != 0:
            raise RuntimeError("compile failed: " + " ".join(cmd))
    link = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.run(link, check=True)
    os.replace(LIB + ".tmp", LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
