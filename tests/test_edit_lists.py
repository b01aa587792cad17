"""Overlap lists are made for the edit lists whose kernel reads them, and for
no others (tests/c/edit_lists.cpp, on the CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_edit_lists(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    csrc = os.path.join(ROOT, "paper_2608_17390_amd", "csrc")
    exe = str(tmp_path / "edit_lists")
    subprocess.check_call(["g++", "-O1", "-g", "-fsanitize=address,undefined", "-std=c++17", "-pthread",
                           "-I" + os.path.join(ROOT, "include"), "-I" + csrc, "-o", exe,
                           os.path.join(ROOT, "tests", "c", "edit_lists.cpp"),
                           os.path.join(csrc, "tc_plan.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.endswith("0 failures\n"), r.stdout + r.stderr
