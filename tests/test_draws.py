"""The FP32 form of a physics draw stays within the margin that its use allows
(1.9e-7 in log2: half an ulp of FP32 for each of its two roundings, times
log2(e), and a little), down to the smallest draw, 2^-54.  Host code only."""
import os
import subprocess

from paper_1512_06637_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fp32_draw_within_margin(tmp_path):
    exe = tmp_path / "draw_check"
    cmd = [build.hipcc(), "-O1", "-std=c++17", "-w", "--cuda-host-only", os.path.join(HERE, "native", "draw_check.hip"),
           "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
