"""Which chunks of columns a wide product goes through in: on both sides of the rule's lines, the same sums."""
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


@pytest.mark.parametrize("k", [255, 256, 257, 301, 320, 384, 385, 500, 513, 640, 700])
def test_wide_products(env, k):
    torch, cbm = env
    g = wl.make_graph("citation", n=1500, p_in=5e-3, p_out=3e-4)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, max_depth=1)
    X = wl.integer_features(g.n, k, 3)
    Y = torch.full((g.n, k), float("nan"), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(g.rowptr, g.colidx, X))


@pytest.mark.parametrize("n,ks", [((1 << 20) - 1, (192,)), (1 << 20, (192, 128, 320)), (1953124, (128,)), (1953125, (128, 124)), (1 << 21, (128, 192, 256))])
def test_slabs_of_64_columns_of_a_large_x(env, n, ks):
    """Node i and its neighbours i - 1 and i + 1 on a ring, and node 0 with 300 more (a split row): sums of three whole numbers."""
    torch, cbm = env
    nodes = np.arange(n, dtype=np.int64)
    more = 1000 + 7 * np.arange(300, dtype=np.int64)
    rowptr, colidx = wl.graphs.csr_from_edges(n, np.concatenate((nodes, np.zeros(300, np.int64))), np.concatenate(((nodes + 1) % n, more)))
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    at = torch.from_numpy(more).cuda()
    for k in ks:
        X = torch.randint(-8, 9, (n, k), device="cuda", generator=torch.Generator(device="cuda").manual_seed(k)).float()
        Y = torch.full_like(X, float("nan"))
        cbm.cbm_spmm(h, X, Y)
        want = torch.roll(X, 1, 0).add_(torch.roll(X, -1, 0))
        want[0] += X[at].sum(0)
        want[at] += X[0]
        assert torch.equal(Y, want), k


@pytest.mark.parametrize("n,shuffled", [(16383, False), (16384, False), (70001, False), (20000, True)])
def test_rows_shared_out_in_their_own_order(env, capfd, monkeypatch, n, shuffled):
    """Rows whose neighbours in the matrix hold the same columns go to the XCDs in contiguous shares; every row is written once, whatever their order."""
    torch, cbm = env
    monkeypatch.setenv("CBM_VERBOSE", "1")
    rng = np.random.default_rng(n)
    src = rng.integers(0, n, 3 * n)
    dst = np.clip(src + rng.integers(-40, 41, 3 * n), 0, n - 1)
    if shuffled:
        label = rng.permutation(n)
        src, dst = label[src], label[dst]
    rowptr, colidx = wl.graphs.csr_from_edges(n, src, dst)
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    said = [ln.split() for ln in capfd.readouterr().err.splitlines() if "columns on an XCD" in ln]
    assert len(said) == (n >= 16384) and all((int(s[5]) <= 0.9 * int(s[12])) != shuffled for s in said)
    for k in (5, 64, 200):
        X = wl.integer_features(n, k, 3)
        Y = torch.full((n, k), float("nan"), device="cuda")
        cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, X))
        if k == 64:
            cbm.cbm_profile_enable(h, True)
            cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
            torch.cuda.synchronize()
            assert [r["per_xcd"] for r in cbm.cbm_profile_read(h)] == [int(n >= 16384 and not shuffled)]
            cbm.cbm_profile_enable(h, False)
