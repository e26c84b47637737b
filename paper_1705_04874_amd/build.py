"""Build the HIP library paper_1705_04874_amd/libpstd3d.so for gfx950 with hipcc."""
import os
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpstd3d.so")
# (source, object, extra flags): the solver's kernels are compiled per group of
# grid lengths, side by side (pstd_variants.hpp)
SOURCES = [("pstd_variants.hip", f"pstd_variants_{g}.o", [f"-DPSTD_GROUP={g}"]) for g in range(8)]
SOURCES += [(s, s + ".o", []) for s in ("sno.hip", "combine.hip", "pstd3d.hip", "catalog.hip")]

# Packed FP32 instructions are disabled for every HIP translation unit.
HIPFLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose=True, jobs=None):
    objs = []
    t0 = time.time()
    procs = []
    for s, o, flags in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(CSRC, o)
        cmd = ["hipcc", "-c"] + HIPFLAGS + flags + ["-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((subprocess.Popen(cmd), cmd))
        objs.append(obj)
    for p, cmd in procs:
        if p.wait() != 0:
            raise RuntimeError("compile failed: " + " ".join(cmd))
    tmp = LIB + ".tmp"
    cmd = ["hipcc", "-shared", "--offload-arch=gfx950", "-o", tmp] + objs
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB} in {time.time() - t0:.0f}s", flush=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
