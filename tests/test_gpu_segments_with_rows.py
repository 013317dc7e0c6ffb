"""Segments of split rows and rows stored in full in one launch: the bits of the two launches apart (which per-launch times still take), and the sums."""
import numpy as np
import pytest

import workloads as wl
from oracle import cbm_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2409_02208_amd as cbm

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch, cbm


def _graph(kind):
    if kind == "rmat":
        g = wl.make_graph("rmat", scale=12, edge_factor=24)
        return g.n, g.rowptr, g.colidx
    # neighbours in the matrix that share columns (contiguous shares of rows for each XCD), and a few rows of hundreds of entries
    n = 20000
    rng = np.random.default_rng(5)
    src = rng.integers(0, n, 3 * n)
    dst = np.clip(src + rng.integers(-40, 41, 3 * n), 0, n - 1)
    hubs = rng.integers(0, n, 5)
    src, dst = np.concatenate((src, np.repeat(hubs, 700))), np.concatenate((dst, rng.integers(0, n, 3500)))
    return (n, *wl.graphs.csr_from_edges(n, src, dst))


@pytest.mark.parametrize("hubs", ["0", "2"])
@pytest.mark.parametrize("kind", ["rmat", "shares"])
def test_one_launch_gives_what_two_give(env, monkeypatch, kind, hubs):
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", "0")  # (not the launch of small products)
    monkeypatch.setenv("CBM_HUB_BLOCKS", hubs)
    monkeypatch.setenv("CBM_ROW_BLOCKS", "0")
    monkeypatch.setenv("CBM_SHARED_SUMS", "0")
    n, rowptr, colidx = _graph(kind)
    for loops in (False, True):
        h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=loops, max_depth=0 if hubs == "2" else 1)
        assert cbm.cbm_stats(h)["num_split_rows"] > 0
        calls = [lambda X, Y: cbm.cbm_spmm(h, X, Y), lambda X, Y: cbm.cbm_spmm_mean(h, X, Y), lambda X, Y: cbm.cbm_spmm_gin(h, 0.25, X, Y)]
        if loops:
            calls += [lambda X, Y: cbm.cbm_spmm_normalized(h, X, Y), lambda X, Y: cbm.cbm_spmm_normalized_relu(h, X, Y)]
        # widths of 8, 16, 32 and 64 lanes, one chunk of columns and several, whole lines and odd strides
        for k, ld in ((1, 1), (8, 8), (47, 47), (64, 64), (100, 104), (128, 128), (200, 200), (256, 256), (300, 301)):
            gen = torch.Generator(device="cuda").manual_seed(k)
            X = torch.randn(n, ld, device="cuda", generator=gen)[:, :k]
            for call in calls:
                got, want = (torch.full((n, k), float("nan"), device="cuda") for _ in range(2))
                call(X, got)
                cbm.cbm_profile_enable(h, True)
                call(X, want)
                torch.cuda.synchronize()
                kinds = [r["kind"] for r in cbm.cbm_profile_read(h)]
                cbm.cbm_profile_enable(h, False)
                assert 0 in kinds and 1 in kinds  # rows and segments, each a launch
                assert torch.equal(got, want), (k, loops)
        X = wl.integer_features(n, 36, 1)
        Y = torch.full((n, 36), float("nan"), device="cuda")
        cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
        ref = orc.spmm_csr(rowptr, colidx, X) + (X if loops else 0)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
