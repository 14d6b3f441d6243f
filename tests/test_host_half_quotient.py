"""The two-operation quotient of 16-bit weights is the IEEE quotient (host check, exhaustive)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_all_significands(tmp_path):
    exe = str(tmp_path / "host_half_quotient")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "paper_2202_07471_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host_half_quotient.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, check=True)
    assert "half_quotients=7340032 mismatches=0" in out.stdout
