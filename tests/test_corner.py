"""The single-precision walk's step where rounding leaves it open, against a
walk in whole numbers (tests/c/corner_check.cpp), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("seed", [1, 2])
def test_corner_steps(tmp_path, seed):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "corner_check")
    # (no contraction: the products and sums of the step round one by one)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off",
                           "-I" + os.path.join(ROOT, "paper_2608_17390_amd", "csrc"), "-o", exe,
                           os.path.join(ROOT, "tests", "c", "corner_check.cpp")])
    r = subprocess.run([exe, "150000", str(seed)], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout
