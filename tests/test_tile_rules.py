"""The rules that choose a product's tiles, on the CPU: tests/rule_check.cpp, built with g++ against tilerule.hpp."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_01464_amd", "csrc")


def test_tile_rules(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    exe = str(tmp_path / "rule_check")
    cmd = [gxx, "-std=c++17", "-O1", f"-I{CSRC}", os.path.join(HERE, "rule_check.cpp"), "-o", exe]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "rules ok" in r.stdout, r.stderr[-4000:]
