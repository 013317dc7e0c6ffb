"""The grid of dense products with B in registers, where several panels of columns lie side by side."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_no_workgroup_waits_for_others_to_end(tmp_path):
    exe = str(tmp_path / "harness")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2409_02208_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_panel_blocks_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "panel blocks ok" in r.stdout, r.stdout
