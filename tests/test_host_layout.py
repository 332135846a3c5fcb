"""The index arithmetic that the packing of the operators and the kernels that
read them share, at axes so long that 32 bits do not hold it.  No GPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_operator_blocks_of_long_axes(tmp_path):
    exe = str(tmp_path / "layout_check")
    cmd = ["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
           os.path.join(ROOT, "tests", "host", "layout_check.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and "layout checks ok" in run.stdout, run.stdout + run.stderr
