"""build.py takes the offload architecture from GV_OFFLOAD_ARCH: the physics
draws, which use an instruction that only gfx950 has, compile for gfx942 too."""
import subprocess

import pytest

from paper_1512_06637_amd import build

SRC = """#include <hip/hip_runtime.h>
#include "gv_phys.h"
__global__ void k(gv::CQ rate, double* out, int* proc) {
  out[threadIdx.x] = gv::physics_length(rate, 3, 0, 5, threadIdx.x, 1, proc + threadIdx.x);
}
"""


@pytest.mark.parametrize("arch", ["gfx942", "gfx950"])
def test_draws_compile(arch, tmp_path):
    src = tmp_path / "draws.hip"
    src.write_text(SRC)
    cmd = [build.hipcc(), f"--offload-arch={arch}", "-O1", "-std=c++17", "-w", "--cuda-device-only",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", build.CSRC, "-c", str(src),
           "-o", str(tmp_path / "draws.o")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
