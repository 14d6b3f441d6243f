"""The launch shapes of 1x1 / FC rows cover every row (host check)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_row_is_covered(tmp_path):
    exe = str(tmp_path / "host_launch_shape_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2202_07471_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host_launch_shape_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, check=True)
    assert "shape_mismatches=0" in out.stdout
