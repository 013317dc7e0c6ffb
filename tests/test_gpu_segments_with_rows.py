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
    # neighbours in the matrix that share columns (contiguous shares of rows for each XCD), and a few rows of hundreds of entries, half of them the same
    n = 20000
    rng = np.random.default_rng(5)
    src = rng.integers(0, n, 3 * n)
    dst = np.clip(src + rng.integers(-40, 41, 3 * n), 0, n - 1)
    hubs = rng.integers(0, n, 5)
    src = np.concatenate((src, np.repeat(hubs, 700)))
    dst = np.concatenate((dst, np.concatenate([np.concatenate((np.arange(350) * 50, rng.integers(0, n, 350))) for _ in hubs])))
    return (n, *wl.graphs.csr_from_edges(n, src, dst))


def _records(torch, cbm, h, on, call):
    cbm.cbm_profile_enable(h, on)
    call()
    torch.cuda.synchronize()
    records = cbm.cbm_profile_read(h)
    cbm.cbm_profile_enable(h, 0)
    return records


def _calls(cbm, h, loops):
    calls = [lambda X, Y: cbm.cbm_spmm(h, X, Y), lambda X, Y: cbm.cbm_spmm_mean(h, X, Y), lambda X, Y: cbm.cbm_spmm_gin(h, 0.25, X, Y)]
    if loops:
        calls += [lambda X, Y: cbm.cbm_spmm_normalized(h, X, Y), lambda X, Y: cbm.cbm_spmm_normalized_relu(h, X, Y)]
    return calls


def _one_launch_gives_what_two_give(torch, cbm, h, n, k, ld, call, hubs):
    gen = torch.Generator(device="cuda").manual_seed(k)
    X = torch.randn(n, ld, device="cuda", generator=gen)[:, :k]
    got, timed, want = (torch.full((n, k), float("nan"), device="cuda") for _ in range(3))
    call(X, got)
    one = _records(torch, cbm, h, 2, lambda: call(X, timed))
    two = _records(torch, cbm, h, 1, lambda: call(X, want))
    first = [5] if hubs else []
    assert [r["kind"] for r in one] == first + [7, 2] and [r["kind"] for r in two] == first + [1, 0, 2], k
    one, two = one[len(first)], two[len(first):]
    for what in ("tasks", "deltas", "algorithmic_bytes"):
        assert one[what] == two[0][what] + two[1][what]
    assert torch.equal(got, want) and torch.equal(timed, want), k
    return one


@pytest.mark.parametrize("hubs", ["0", "2"])
@pytest.mark.parametrize("kind", ["rmat", "shares"])
def test_one_launch_gives_what_two_give(env, monkeypatch, kind, hubs):
    torch, cbm = env
    for name, value in (("FLAT_WAVES", "0"), ("ROW_BLOCKS", "0"), ("SHARED_SUMS", "0"), ("HUB_BLOCKS", hubs)):  # (none of the other ways of a product)
        monkeypatch.setenv("CBM_" + name, value)
    n, rowptr, colidx = _graph(kind)
    for loops in (False, True):
        h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=loops, max_depth=0 if hubs == "2" else 1)
        assert cbm.cbm_stats(h)["num_split_rows"] > 0
        # widths of 8, 16, 32 and 64 lanes, one chunk of columns and several, whole lines and odd strides
        for k, ld in ((1, 1), (8, 8), (47, 47), (64, 64), (100, 104), (128, 128), (200, 200), (256, 256), (300, 301)):
            for call in _calls(cbm, h, loops):
                _one_launch_gives_what_two_give(torch, cbm, h, n, k, ld, call, hubs == "2")
        X = wl.integer_features(n, 36, 1)
        Y = torch.full((n, 36), float("nan"), device="cuda")
        cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
        ref = orc.spmm_csr(rowptr, colidx, X) + (X if loops else 0)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("hubs", ["0", "2"])
def test_one_launch_of_many_work_items(env, monkeypatch, hubs):
    """From 65,536 waves on the launch is the build of the kernel that takes rows of X two at a time."""
    torch, cbm = env
    for name, value in (("FLAT_WAVES", "0"), ("ROW_BLOCKS", "0"), ("SHARED_SUMS", "0"), ("HUB_BLOCKS", hubs)):  # (none of the other ways of a product)
        monkeypatch.setenv("CBM_" + name, value)
    n, rng = 300000, np.random.default_rng(9)
    src, dst = rng.integers(0, n, (2, 4 * n))
    long = rng.integers(0, n, 6).repeat(900)
    src, dst = np.concatenate((src, long)), np.concatenate((dst, np.concatenate([np.concatenate((np.arange(400) * 700, rng.integers(0, n, 500))) for _ in range(6)])))
    rowptr, colidx = wl.graphs.csr_from_edges(n, src, dst)
    for loops in (False, True):
        h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=loops, max_depth=0)
        for k, ld, group in ((47, 47, 4), (64, 64, 4), (100, 104, 2), (250, 250, 1)):
            for call in _calls(cbm, h, loops):
                record = _one_launch_gives_what_two_give(torch, cbm, h, n, k, ld, call, hubs == "2")
                assert record["tasks"] // group >= 65536
        X = wl.integer_features(n, 36, 1)
        Y = torch.full((n, 36), float("nan"), device="cuda")
        cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
        ref = orc.spmm_csr(rowptr, colidx, X) + (X if loops else 0)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
