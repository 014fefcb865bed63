"""The host copy's second thread: a failure to get one stays inside."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_both_parts_run_whatever_becomes_of_the_second_thread(tmp_path):
    exe = str(tmp_path / "two_threads")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_1607_05535_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "two_threads_driver.cpp"), "-o", exe],
                   check=True, capture_output=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
