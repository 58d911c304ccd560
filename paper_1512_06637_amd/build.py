"""Builds libgvgeom.so (the HIP library behind include/gvgeom.h) for gfx950, in-tree."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgvgeom.so")
SOURCES = ["gv_inst_lane_phys64.hip", "gv_inst_lane_phys32.hip", "gv_inst_lane.hip", "gv_inst_lane_nav64.hip",
           "gv_inst_lane_nav32.hip", "gv_inst_step.hip", "gv_inst_step_phys.hip", "gv_inst_lane_composites.hip",
           "gv_inst_query.hip", "gv_abi.hip"]
ARCH = os.environ.get("GV_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for c in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), "hipcc"):
        if os.path.sep not in c or os.path.exists(c):
            return c
    return "hipcc"


def build(verbose: bool = False) -> str:
    """Compiles every source (in parallel) and links the library."""
    flags = [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
             # no packed FP32 instructions in device code
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wall", "-Wno-unused-function", "-Wno-unknown-pragmas"]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(min(8, len(os.sched_getaffinity(0)))) as pool:
            list(pool.map(lambda so: run([hipcc(), *flags, "-c", "-o", so[1], os.path.join(CSRC, so[0])]),
                          zip(SOURCES, objs)))
        run([hipcc(), f"--offload-arch={ARCH}", "-shared", "-o", LIB + ".tmp", *objs])
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
