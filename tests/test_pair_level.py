"""How a pair's tiles are shared out (csrc/pair_level.h, host only)."""
import os
import shutil
import subprocess

import pytest

TESTS = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(TESTS), "paper_2505_14669_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_extra_rounds_are_the_best_of_all(tmp_path):
    program = str(tmp_path / "check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, os.path.join(TESTS, "hostcheck", "pair_level_check.cpp"), "-o", program], check=True)
    r = subprocess.run([program], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
