"""Builds the HIP-free plan of the register-window refocus with g++ (address
and undefined-behaviour sanitizers) and runs its host tests."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_20692_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_window_plan_with_sanitizers(tmp_path):
    exe = str(tmp_path / "window_test")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", CSRC, os.path.join(CSRC, "refocus_window_plan.cpp"),
           os.path.join(ROOT, "tests", "host", "window_test.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert "window tests passed" in r.stdout
