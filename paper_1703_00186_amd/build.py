"""Builds the gfx950 shared library behind include/lb.h.

    python -m paper_1703_00186_amd.build

compiles csrc/*.hip with hipcc for gfx950 into paper_1703_00186_amd/libd2q37_lb.so
(in-tree).  Packed-FP32 VALU instructions are disabled for all device code.
"""

from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libd2q37_lb.so")
SOURCES = ["d2q37_kernels.hip", "d2q37_coeff.hip", "d2q37_pair.hip", "d2q37_variants.hip",
           "lb_api.hip", "lb_scratch.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]
# The marching kernels without loop-invariant code motion on machine code: it
# moves some 120 FP64 literals out of their loops, which then are spilled and
# read back lane by lane (266 spilled scalars in the double plain BGK step, 24
# without).  The site kernels keep it: without, the FP32 observables of 512 x 512
# take 29.5 us instead of 28.9.
MARCHING = {"d2q37_coeff.hip", "d2q37_pair.hip"}
MARCHING_FLAGS = ["-mllvm", "-disable-machine-licm"]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = False) -> str:
    sys.path.insert(0, CSRC)
    try:
        import gen_constants
    finally:
        sys.path.pop(0)
    if not gen_constants.check():
        gen_constants.write()
    tmp = LIB + ".tmp%d" % os.getpid()

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as objects:
        def compile_one(name):
            out = os.path.join(objects, name + ".o")
            run([hipcc()] + HIPCC_FLAGS + (MARCHING_FLAGS if name in MARCHING else [])
                + ["-c", os.path.join(CSRC, name), "-o", out])
            return out

        with concurrent.futures.ThreadPoolExecutor(max_workers=4) as pool:
            built = list(pool.map(compile_one, SOURCES))
        run([hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared"] + built + ["-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
