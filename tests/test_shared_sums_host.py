"""Shared sums on the host: sets and rows add up to the matrix, tree and counters stay as they are, the automatic rule takes them where it should."""
import shutil

import numpy as np
import pytest

import paper_2409_02208_amd as cbm
import workloads as wl
from test_row_blocks_host import SANITIZED, _harness


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_sets_and_rows_add_up_to_the_matrix(tmp_path):
    assert "sums ok" in _harness(tmp_path, "host_sums_main.cpp", *SANITIZED)


def test_sums_leave_tree_and_counters_alone(monkeypatch):
    g = wl.make_graph("collaboration", n=6000)
    handles = []
    for want in ("0", "1"):
        monkeypatch.setenv("CBM_SHARED_SUMS", want)
        handles.append(cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True, host_only=True))
    a, b = (cbm.cbm_stats(h) for h in handles)
    assert {k: v for k, v in a.items() if k != "build_seconds"} == {k: v for k, v in b.items() if k != "build_seconds"}
    for x, y in zip(cbm.cbm_get_tree(handles[0]).values(), cbm.cbm_get_tree(handles[1]).values()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("name,kw,taken", [("collaboration", dict(n=20000), True), ("citation", dict(n=5000, p_in=1.6e-3, p_out=8e-5), False),
                                           ("protein", dict(n=4000, knn=60), False), ("rmat", dict(scale=13), False)])
def test_who_takes_shared_sums(monkeypatch, capfd, name, kw, taken):
    monkeypatch.setenv("CBM_SHARED_SUMS", "2")
    monkeypatch.setenv("CBM_ROW_BLOCKS", "2")
    monkeypatch.setenv("CBM_HUB_BLOCKS", "3")
    monkeypatch.setenv("CBM_VERBOSE", "1")
    g = wl.make_graph(name, **kw)
    cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True, host_only=True)
    said = [ln for ln in capfd.readouterr().err.splitlines() if "shared sums" in ln and "products" in ln]
    assert len(said) == 1 and ("products take them" in said[0]) == taken
