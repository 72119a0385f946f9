"""The fp64 exponential of the one-pass evaluation of a rejected row, compiled for the host from the device's header."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def figures(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("exp_units") / "exp_units_check")
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_2410_03355_amd", "csrc"),
                    os.path.join(ROOT, "tests", "exp_units_check.cpp"), "-o", exe, "-lquadmath", "-lm"], check=True)
    return [float(x) for x in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split()]


def test_exp_units_within_one_rounding(figures):
    """Half a unit in the last place for the last step; below it the polynomial's 6e-18 (0.03 units) and the rounding
    of the smaller terms (0.02)."""
    worst, differ, ends = figures[:3]
    assert worst <= 0.55
    assert differ == 0 and ends == 1


def test_exp_units_nonpos(figures):
    """The same where the result is a normal number; below, where it is rounded once more, a little over half a unit of
    the smallest number.  Differences from a maximum of any size: what lies far below it is nothing."""
    worst, below, wrong = figures[3:6]
    assert worst <= 0.55
    assert below <= 1.0
    assert wrong == 0


def test_exp_units_any_far_from_zero(figures):
    """Logits down to 1100 below a reference of 4096 in magnitude: the same bounds."""
    worst, below = figures[6:]
    assert worst <= 0.55
    assert below <= 1.0
