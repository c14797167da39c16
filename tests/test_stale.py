"""Hooks that decide on a cached copy of the shadow word: a compiled check over
random histories of one word compares the outcome with the pairwise
definition, whatever earlier state each load returned."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2401_04701_amd", "csrc")


def test_stale_loads_find_the_same_races(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "stale_check")
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "stale_check.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert all(int(n) > 10000 for n in r.stdout.split())
