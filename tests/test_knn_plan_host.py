"""Every candidate list that the neighbour table's plan allows is held whole by the selection kernel it gets."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_selection_holds_the_longest_list(tmp_path):
    exe = tmp_path / "knn_plan_check"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2410_03355_amd", "csrc"),
                    os.path.join(ROOT, "tests", "knn_plan_check.cpp"), "-o", str(exe)], check=True)
    keys, tokens, narrow_long, keys_large, *kernels, lost = map(int, subprocess.run([str(exe)], check=True, capture_output=True,
                                                                                    text=True).stdout.split())
    assert keys > 1000 and tokens > 1000
    assert narrow_long > 100 and keys_large > 100     # the grid covers long lists of narrow tables
    assert all(n > 100 for n in kernels)              # and every kernel that ranks lists of tokens
    assert lost == 0
