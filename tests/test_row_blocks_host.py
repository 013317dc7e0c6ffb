"""Row blocks on the host: the blocks decode to the matrix, and the automatic policy leaves the tree and its counters alone."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import paper_2409_02208_amd as cbm
import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_blocks_decode_to_the_matrix(tmp_path):
    exe = str(tmp_path / "host_blocks")
    csrc = os.path.join(ROOT, "paper_2409_02208_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"),
           "-I", csrc, os.path.join(ROOT, "tests", "host_blocks_main.cpp"), os.path.join(csrc, "cbm_builder.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0 and "sanitize" in r.stderr:
        pytest.skip("sanitizer runtime not available: " + r.stderr[-200:])
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "blocks ok" in r.stdout and "hubs ok" in r.stdout, (r.stdout[-500:], r.stderr[-3000:])


def test_blocks_leave_tree_and_counters_alone(monkeypatch):
    g = wl.make_graph("protein", n=3000, knn=40)
    handles = []
    for want in ("0", "1"):
        monkeypatch.setenv("CBM_ROW_BLOCKS", want)
        handles.append(cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True, host_only=True))
    a, b = (cbm.cbm_stats(h) for h in handles)
    assert {k: v for k, v in a.items() if k != "build_seconds"} == {k: v for k, v in b.items() if k != "build_seconds"}
    for x, y in zip(cbm.cbm_get_tree(handles[0]).values(), cbm.cbm_get_tree(handles[1]).values()):
        assert np.array_equal(x, y)
