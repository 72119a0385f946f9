"""The short fp64 exponential for non-positive arguments gives the general one's values, bit for bit."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_short_exponential_equals_the_general_one(tmp_path):
    exe = tmp_path / "exp64_nonpos_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-I",
                    os.path.join(ROOT, "paper_2410_03355_amd", "csrc"),
                    os.path.join(ROOT, "tests", "exp64_nonpos_check.cpp"), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split() == ["0"]
