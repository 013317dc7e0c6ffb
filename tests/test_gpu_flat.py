"""Small products of rows stored in full, a wave or a group of lanes for each row, against the oracle and against the launches that larger products
take: row lengths and widths around the edges, every epilogue, strided and misaligned operands, rows that are split, the choice beside row blocks."""
import numpy as np
import pytest

import workloads as wl
from oracle import cbm_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2409_02208_amd as cbm

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch, cbm


def _err(got, ref, scale_from=None):
    d = np.abs(got.astype(np.float64) - ref).max(axis=1)
    s = np.abs(ref if scale_from is None else scale_from).max(axis=1)
    assert np.all(d[s == 0] == 0)
    return float((d[s > 0] / s[s > 0]).max()) if np.any(s > 0) else 0.0


def _lengths(n, lengths, seed):
    rng = np.random.default_rng(seed)
    rows = [np.sort(rng.choice(n, size=min(n, int(ln)), replace=False)) for ln in lengths]
    rowptr = np.concatenate(([0], np.cumsum([len(r) for r in rows]))).astype(np.int64)
    return rowptr, np.concatenate(rows).astype(np.int32)


@pytest.fixture(scope="module")
def square():
    edges = [0, 1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 130, 200, 511, 512, 513, 700]
    return _lengths(701, (edges * 40)[:701], 1)


@pytest.mark.parametrize("waves", ["0", "100000"])
@pytest.mark.parametrize("k", [1, 4, 8, 31, 32, 33, 47, 64, 65, 100, 128, 129, 200, 256, 260, 500])
def test_sums_of_whole_numbers_are_exact(env, monkeypatch, square, k, waves):
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", waves)
    rowptr, colidx = square
    n = len(rowptr) - 1
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    X = wl.integer_features(n, k, 3)
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((n, k), float("nan"), device="cuda")
    ref = orc.spmm_csr(rowptr, colidx, X)
    cbm.cbm_spmm(h, Xd, Y)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
    cbm.cbm_spmm_noalloc(h, Xd, Y.fill_(float("nan")))
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("lengths,m,n", [([5000] * 3, 3, 9000), ([0] * 50, 50, 7), ([40] * 9, 9, 60), ([3] * 1000 + [900], 1001, 1000), ([129, 0, 0, 5], 4, 300)])
def test_few_rows_of_one_kind(env, monkeypatch, lengths, m, n):
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", "100000")
    rowptr, colidx = _lengths(n, lengths, 2)
    h = cbm.cbm_build(m, n, rowptr, colidx, max_depth=1)
    for k in (3, 64, 150):
        X = wl.integer_features(n, k, 4)
        Y = torch.full((m, k), float("nan"), device="cuda")
        cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, X))


@pytest.mark.parametrize("layout", ["dense", "strided", "misaligned"])
@pytest.mark.parametrize("k", [16, 47, 128, 160])
def test_every_epilogue(env, monkeypatch, square, k, layout):
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", "100000")
    rowptr, colidx = square
    n = len(rowptr) - 1
    hn = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, max_depth=1)
    ht = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, max_depth=1, transpose=True)
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    X = wl.gaussian_features(n, k, 5)
    pad, off = {"dense": (0, 0), "strided": (5, 0), "misaligned": (4, 1)}[layout]
    Xd = torch.zeros((n, k + pad), device="cuda")[:, off:off + k]
    Xd.copy_(torch.from_numpy(X))
    room = torch.full((n, k + pad), float("nan"), device="cuda")
    Y = room[:, off:off + k]

    def run(fn, *args):
        room.fill_(float("nan"))
        fn(*args, Xd, Y)
        torch.cuda.synchronize()
        got = room.cpu().numpy()
        assert np.isnan(np.delete(got, np.arange(off, off + k), axis=1)).all(), "wrote outside the columns"
        return got[:, off:off + k]

    norm = orc.spmm_csr_normalized(rowptr, colidx, X)
    plain = orc.spmm_csr(rowptr, colidx, X)
    assert _err(run(cbm.cbm_spmm_normalized, hn), norm) <= TOL
    assert _err(run(cbm.cbm_spmm_normalized_relu, hn), np.maximum(norm, 0), norm) <= TOL
    assert _err(run(cbm.cbm_spmm_mean, h), orc.spmm_csr_mean(rowptr, colidx, X)) <= TOL
    assert _err(run(cbm.cbm_spmm_gin, h, 0.5), plain + 1.5 * X.astype(np.float64)) <= TOL
    assert _err(run(cbm.cbm_spmm, h), plain) <= TOL
    Z = run(cbm.cbm_spmm_normalized, ht).astype(np.float64)
    G = wl.gaussian_features(n, k, 6).astype(np.float64)
    ref = orc.spmm_csr_normalized(rowptr, colidx, G.astype(np.float32))
    assert abs((ref * X).sum() - (G * Z).sum()) <= 1e-5 * np.abs(ref * X).sum()


def test_segments_and_rows_in_one_launch_or_two(env, monkeypatch, square):
    """With profiling on they are launched apart; either way every work item is counted, and the sums are the same bit for bit."""
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", "100000")
    rowptr, colidx = square
    n = len(rowptr) - 1
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, max_depth=1)
    assert cbm.cbm_stats(h)["num_split_rows"] > 0
    X = torch.from_numpy(wl.gaussian_features(n, 72, 1)).cuda()
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    cbm.cbm_spmm_normalized(h, X, Y)
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm_normalized(h, X, Z)
    torch.cuda.synchronize()
    recs = cbm.cbm_profile_read(h)
    assert [r["kind"] for r in recs] == [1, 0, 2] and sum(r["tasks"] for r in recs[:2]) == cbm.cbm_stats(h)["num_tasks"]
    assert torch.equal(Y, Z)


def test_infinities_and_nan_stay_in_their_rows(env, monkeypatch, square):
    torch, cbm = env
    monkeypatch.setenv("CBM_FLAT_WAVES", "100000")
    rowptr, colidx = square
    n, k = len(rowptr) - 1, 40
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    X = wl.integer_features(n, k, 8)
    X[3, 0], X[700, 33], X[41, 5], X[42, 5], X[600, 39] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    with np.errstate(invalid="ignore"):
        ref = np.stack([X[colidx[a:b]].sum(0) if b > a else np.zeros(k) for a, b in zip(rowptr[:-1], rowptr[1:])])
    Y = torch.empty((n, k), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
    assert np.array_equal(Y.cpu().numpy(), ref.astype(np.float32), equal_nan=True)


@pytest.mark.parametrize("name,kw,narrow,wide", [("tiny", {}, [0], [0]), ("protein", dict(n=4000, knn=60), [0], [5]), ("collaboration", dict(n=12000), [0], [6, 6]),
                                                ("citation", dict(n=4000, p_in=2e-3, p_out=1e-4), [0], [0])])
def test_which_launches_a_small_product_takes(env, name, kw, narrow, wide):
    """Row blocks and shared sums stand back where the rows as they are take less: the device holds both, and the width decides."""
    torch, cbm = env
    g = wl.make_graph(name, **kw)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    for k, kinds in ((16, narrow), (256, wide)):
        X = wl.gaussian_features(g.n, k, 1)
        Xd, Y, Z = torch.from_numpy(X).cuda(), torch.empty((g.n, k), device="cuda"), torch.empty((g.n, k), device="cuda")
        cbm.cbm_spmm_normalized(h, Xd, Y)
        assert _err(Y.cpu().numpy(), orc.spmm_csr_normalized(g.rowptr, g.colidx, X)) <= TOL
        cbm.cbm_spmm(h, Xd, Y)
        cbm.cbm_spmm_noalloc(h, Xd, Z)
        assert torch.equal(Y, Z)
        cbm.cbm_profile_enable(h, True)
        cbm.cbm_spmm_normalized(h, Xd, Y)
        torch.cuda.synchronize()
        assert [r["kind"] for r in cbm.cbm_profile_read(h)] == kinds, (k, kinds)
        cbm.cbm_profile_enable(h, False)


def test_the_environment_is_read_when_the_handle_is_built(env, monkeypatch, square):
    torch, cbm = env
    rowptr, colidx = square
    n = len(rowptr) - 1
    X = torch.from_numpy(wl.gaussian_features(n, 32, 1)).cuda()
    Y, Z, want = (torch.empty_like(X) for _ in range(3))
    h = cbm.cbm_build(n, n, rowptr, colidx, max_depth=1)
    cbm.cbm_spmm(h, X, want)
    monkeypatch.setenv("CBM_FLAT_WAVES", "0")
    cbm.cbm_spmm(h, X, Y)
    cbm.cbm_spmm(cbm.cbm_build(n, n, rowptr, colidx, max_depth=1), X, Z)   # the kernels that larger products take: other orders of addition
    assert torch.equal(Y, want) and not torch.equal(Z, want)
