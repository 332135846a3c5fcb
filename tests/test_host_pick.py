"""The request server's choice of the next request: the pass limit and the
window it looks through.  No GPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_oldest_request_is_passed_over_a_bounded_number_of_times(tmp_path):
    exe = str(tmp_path / "pick_check")
    cmd = ["g++", "-std=c++17", "-O1", "-D_GLIBCXX_ASSERTIONS", "-fsanitize=undefined",
           "-fno-sanitize-recover=all", os.path.join(ROOT, "tests", "host", "pick_check.cpp"),
           "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "pick checks ok" in run.stdout, run.stdout + run.stderr
