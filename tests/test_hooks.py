"""The hooks as their steps interleave: a compiled model with loads that return
any earlier state of the word (also of an earlier launch), updates of several
accesses at once, and other threads' steps between exchange and fold, against
the pairwise definition."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2401_04701_amd", "csrc")


def test_interleaved_hooks_find_the_same_races(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "hook_check")
    subprocess.run([gxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(HERE, "hook_check.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert all(int(n) > 10000 for n in r.stdout.split())
