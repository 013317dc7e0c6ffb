"""Which dense products hold B in registers, against measured ones on both sides of the lines; how many waves share K there."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_the_faster_kernels_are_taken(tmp_path):
    exe = str(tmp_path / "harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2409_02208_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_held_rule_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "held rule ok" in r.stdout, r.stdout
