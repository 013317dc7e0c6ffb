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


@pytest.mark.parametrize("extra,planned", [(0, True), (1500, False)])
def test_a_row_that_no_set_shortens_is_seen_before_the_plan_is_made(monkeypatch, capfd, extra, planned):
    """One node with neighbours all over: the rows of the plan are not split, so the handle keeps its paths, and says so without looking for all sets;
    what a few rows say does not depend on the number of threads."""
    for name in ("CBM_SHARED_SUMS", "CBM_ROW_BLOCKS"):
        monkeypatch.setenv(name, "2")
    monkeypatch.setenv("CBM_HUB_BLOCKS", "3")
    monkeypatch.setenv("CBM_VERBOSE", "1")
    g = wl.make_graph("collaboration", n=20000)
    src = np.concatenate([np.repeat(np.arange(g.n), np.diff(g.rowptr)), np.full(extra, 7)])
    dst = np.concatenate([g.colidx.astype(np.int64), np.random.default_rng(1).choice(g.n, extra, replace=False)])
    rowptr, colidx = wl.graphs.csr_from_edges(g.n, src[src != dst], dst[src != dst])
    for threads in (1, 3):
        cbm.cbm_build(g.n, g.n, rowptr, colidx, add_self_loops=True, host_only=True, num_threads=threads)
        said = [ln for ln in capfd.readouterr().err.splitlines() if "shared sums:" in ln]
        assert any("sets of" in ln for ln in said) == planned and ("products take them" in said[-1]) == planned
