"""The fp64 exponential of the one-pass evaluation of a rejected row, compiled for the host from the device's header."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exp_units_within_one_rounding(tmp_path):
    """Half a unit in the last place for the last step; below it the polynomial's 6e-18 (0.03 units) and the rounding
    of the smaller terms (0.02)."""
    exe = str(tmp_path / "exp_units_check")
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_2410_03355_amd", "csrc"),
                    os.path.join(ROOT, "tests", "exp_units_check.cpp"), "-o", exe, "-lquadmath", "-lm"], check=True)
    worst, differ, ends = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()
    assert float(worst) <= 0.55
    assert int(differ) == 0 and int(ends) == 1
