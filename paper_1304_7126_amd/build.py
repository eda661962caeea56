"""Build librtm1.so (HIP, gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librtm1.so")
# (object, source, defines); the chemistry kernels build once per radiation
# type and method variant
UNITS = [(f"rt_chem_{r}{v}", "rt_chem.hip", [f"-DRT_CHEM_R={t}", f"-DRT_CHEM_V={v}"])
         for r, t in (("f", "float"), ("d", "double")) for v in range(4)]
UNITS += [(n, n + ".hip", []) for n in ("rt_batch", "rt_transport", "rt_adjoint", "rt_kernels", "rt_api")]

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
    # packed FP32 instructions stay off (hand-checked numerics)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, jobs: int = 0) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = jobs or min(8, os.cpu_count() or 1)

    def compile_unit(unit):
        name, src, defines = unit
        obj = os.path.join(CSRC, name + ".o")
        cmd = [hipcc, *[f for f in HIPCC_FLAGS if f != "-shared"], *defines, "-c", os.path.join(CSRC, src),
               "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(jobs) as pool:
        objs = list(pool.map(compile_unit, UNITS))
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
