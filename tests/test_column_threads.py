"""The shared column check when a thread cannot be started, on the CPU
(tests/c/column_threads.cpp): the answer is the same and the process lives."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_threads_that_cannot_start(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    csrc = os.path.join(ROOT, "paper_2608_17390_amd", "csrc")
    exe = str(tmp_path / "column_threads")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + csrc,
                           "-static-libstdc++", "-Wl,--wrap=pthread_create", "-pthread", "-o", exe,
                           os.path.join(ROOT, "tests", "c", "column_threads.cpp"),
                           os.path.join(csrc, "tc_plan.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout, r.stderr)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout + r.stderr
