"""The columns of row and hub blocks as the device has them: which tiles of a step are not empty."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_active_tiles_are_those_with_bits(tmp_path):
    exe = str(tmp_path / "harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2409_02208_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_active_tiles_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "active tiles ok" in r.stdout, r.stdout
