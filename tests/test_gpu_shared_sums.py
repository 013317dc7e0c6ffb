"""Products through shared sums against the oracle: every epilogue, widths around the lane groups and the chunk of 128 columns, strided and
misaligned operands, values that are not finite, several streams, threads and captures at a time, and the call that allocates nothing."""
import threading

import numpy as np
import pytest

import workloads as wl
from oracle import cbm_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of a row's largest value, as for the paths: sums of 32-bit terms, a row's own column less than ten times over


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2409_02208_amd as cbm

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch, cbm


@pytest.fixture(autouse=True)
def force(monkeypatch):
    monkeypatch.setenv("CBM_SHARED_SUMS", "1")
    monkeypatch.setenv("CBM_ROW_BLOCKS", "0")


def _err(got, ref, scale_from=None):
    d = np.abs(got.astype(np.float64) - ref).max(axis=1)
    s = np.abs(ref if scale_from is None else scale_from).max(axis=1)
    assert np.all(d[s == 0] == 0)
    return float((d[s > 0] / s[s > 0]).max()) if np.any(s > 0) else 0.0


def _kinds(torch, cbm, h, call):
    cbm.cbm_profile_enable(h, True)
    call()
    torch.cuda.synchronize()
    kinds = [r["kind"] for r in cbm.cbm_profile_read(h)]
    cbm.cbm_profile_enable(h, False)
    return kinds


@pytest.fixture(scope="module")
def graph():
    return wl.make_graph("collaboration", n=3000)


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("k", [1, 7, 31, 32, 33, 64, 65, 100, 128, 129, 130, 257, 300])
def test_sums_of_whole_numbers_are_exact(env, graph, k, loops):
    torch, cbm = env
    g = graph
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=loops)
    X = wl.integer_features(g.n, k, 3)
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((g.n, k), float("nan"), device="cuda")
    kinds = _kinds(torch, cbm, h, lambda: cbm.cbm_spmm(h, Xd, Y))
    assert kinds == [6, 6]
    ref = orc.spmm_csr(g.rowptr, g.colidx, X) + (X if loops else 0)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
    cbm.cbm_spmm_noalloc(h, Xd, Y.fill_(float("nan")))
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("layout", ["dense", "strided", "misaligned"])
@pytest.mark.parametrize("k", [16, 47, 96, 128, 160])
def test_every_epilogue(env, graph, k, layout):
    torch, cbm = env
    g = graph
    hn = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx)
    X = wl.gaussian_features(g.n, k, 5)
    pad, off = {"dense": (0, 0), "strided": (5, 0), "misaligned": (4, 1)}[layout]
    Xd = torch.zeros((g.n, k + pad), device="cuda")[:, off:off + k]
    Xd.copy_(torch.from_numpy(X))
    room = torch.full((g.n, k + pad), float("nan"), device="cuda")
    Y = room[:, off:off + k]

    def run(fn, *args):
        room.fill_(float("nan"))
        fn(*args, Xd, Y)
        torch.cuda.synchronize()
        got = room.cpu().numpy()
        assert np.isnan(np.delete(got, np.arange(off, off + k), axis=1)).all(), "wrote outside the columns"
        return got[:, off:off + k]

    norm = orc.spmm_csr_normalized(g.rowptr, g.colidx, X)
    plain = orc.spmm_csr(g.rowptr, g.colidx, X)
    assert _err(run(cbm.cbm_spmm_normalized, hn), norm) <= TOL
    assert _err(run(cbm.cbm_spmm_normalized_relu, hn), np.maximum(norm, 0), norm) <= TOL
    assert _err(run(cbm.cbm_spmm_mean, h), orc.spmm_csr_mean(g.rowptr, g.colidx, X)) <= TOL
    assert _err(run(cbm.cbm_spmm_gin, h, 0.5), plain + 1.5 * X.astype(np.float64)) <= TOL
    assert _err(run(cbm.cbm_spmm_gin, hn, 0.5), plain + 2.5 * X.astype(np.float64)) <= TOL
    assert _err(run(cbm.cbm_spmm, h), plain) <= TOL


def test_directed_graph_and_its_transpose(env):
    """Sets whose rows are not their columns: a directed graph in which groups of nodes point at the same nodes."""
    torch, cbm = env
    rng = np.random.default_rng(4)
    n, k = 1500, 40
    rows = [set() for _ in range(n)]
    for _ in range(200):
        members, also = rng.choice(n, 14, replace=False), rng.choice(n, 3, replace=False)
        for r in members:
            rows[r] |= set(members.tolist()) | set(also.tolist())
    rows = [np.array(sorted(r - {i} if i % 3 else r), dtype=np.int32) for i, r in enumerate(rows)]
    rowptr = np.concatenate(([0], np.cumsum([len(r) for r in rows]))).astype(np.int64)
    colidx = np.concatenate(rows).astype(np.int32)
    X, G = (torch.from_numpy(wl.gaussian_features(n, k, s)).cuda() for s in (1, 2))
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    ht = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, transpose=True)
    assert set(_kinds(torch, cbm, h, lambda: cbm.cbm_spmm_normalized(h, X, Y))) == {6}
    assert set(_kinds(torch, cbm, ht, lambda: cbm.cbm_spmm_normalized(ht, G, Z))) == {6}
    assert _err(Y.cpu().numpy(), orc.spmm_csr_normalized(rowptr, colidx, X.cpu().numpy())) <= TOL
    left, right = float((Y.double() * G.double()).sum()), float((X.double() * Z.double()).sum())
    assert abs(left - right) <= 1e-5 * float((Y.double() * G.double()).abs().sum())


@pytest.mark.parametrize("op", ["normalized", "gin", "spmm", "mean"])
def test_values_that_are_not_finite_are_summed_as_they_stand(env, graph, op):
    """A sum that holds a row's own column more often than the row does is no place for an infinity less itself."""
    torch, cbm = env
    g, k = graph, 50
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=op == "normalized")
    X = wl.gaussian_features(g.n, k, 8)
    X[3, 0], X[700, 33], X[41, 5], X[42, 5], X[900, 49] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    with np.errstate(invalid="ignore"):
        plain = np.add.reduceat(np.vstack([X[g.colidx], np.zeros((1, k))]), np.minimum(g.rowptr[:-1], len(g.colidx)), axis=0).astype(np.float64)
        plain[np.diff(g.rowptr) == 0] = 0
        ref = {"normalized": plain + X, "gin": plain + 1.25 * X, "spmm": plain, "mean": plain}[op]
    Xd, Y = torch.from_numpy(X).cuda(), torch.empty((g.n, k), device="cuda")
    call = {"normalized": cbm.cbm_spmm_normalized, "gin": lambda *a: cbm.cbm_spmm_gin(a[0], 0.25, *a[1:]), "spmm": cbm.cbm_spmm, "mean": cbm.cbm_spmm_mean}[op]
    call(h, Xd, Y)
    torch.cuda.synchronize()
    got = Y.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    clean = np.where(np.isfinite(X), X, 0).astype(np.float32)
    other = torch.empty_like(Y)
    call(h, torch.from_numpy(clean).cuda(), other)
    torch.cuda.synchronize()
    ok = np.isfinite(ref)
    assert np.allclose(got[ok], other.cpu().numpy()[ok], rtol=1e-5, atol=1e-4)


LOWEST = float(np.finfo(np.float32).min)


def _cliques(n, twice=False, size=20, seed=3):
    """Random cliques without self-loops: node i is in 1 + i % 3 of them, or each node in two."""
    rng = np.random.default_rng(seed)
    src, dst = [], []
    for r in range(2 if twice else 3):
        who = rng.permutation(n) if twice else rng.permutation(np.flatnonzero(np.arange(n) % 3 >= r))
        who = who[:len(who) // size * size].reshape(-1, size)
        for i in range(size):
            for j in range(i):
                src.append(who[:, i])
                dst.append(who[:, j])
    return wl.graphs.csr_from_edges(n, np.concatenate(src), np.concatenate(dst))


@pytest.fixture(scope="module")
def cliques():
    return _cliques(3000)


@pytest.mark.parametrize("op", ["spmm", "mean", "gin-1", "gin", "noalloc"])
@pytest.mark.parametrize("k", [16, 50, 128, 160])
def test_a_value_that_its_neighbours_do_not_see(env, cliques, k, op):
    """Sums that hold a row's own value, however large beside its neighbours', leave nothing of it in the row: the error is relative to what the row holds.
    (An own value of up to 32 times the largest other is taken off again: 32 x 2^-24 for each of the few additions that it took part in.)"""
    torch, cbm = env
    rowptr, colidx = cliques
    n = len(rowptr) - 1
    h = cbm.cbm_build(n, n, rowptr, colidx)
    X = wl.gaussian_features(n, k, 9)
    values = (20.0, -40.0, 100.0, 1e3, -1e5, 1e8, -1e20, LOWEST)
    rng = np.random.default_rng(6)
    rows = rng.choice(n, 60, replace=False)       # few of them are neighbours
    for i, r in enumerate(rows):
        X[r, rng.choice(k, 5, replace=False)] = values[i % len(values)]
    X[:, 3] = 0.0                                 # a column that one row alone has anything in, and one of very small values
    X[rows[0], 3] = 0.1
    X[:, 4] *= 1e-41
    X[rows[1], 4] = 1e-30
    s = {"gin-1": 0.0, "gin": 1.25}.get(op)
    call = {"spmm": cbm.cbm_spmm, "mean": cbm.cbm_spmm_mean, "gin-1": lambda *a: cbm.cbm_spmm_gin(a[0], -1.0, *a[1:]),
            "gin": lambda *a: cbm.cbm_spmm_gin(a[0], 0.25, *a[1:]), "noalloc": cbm.cbm_spmm_noalloc}[op]
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((n, k), float("nan"), device="cuda")
    call(h, Xd, Y)
    torch.cuda.synchronize()

    def sums(x):
        out = np.add.reduceat(np.vstack([x[colidx], np.zeros((1, k))]), np.minimum(rowptr[:-1], len(colidx)), axis=0)
        out[np.diff(rowptr) == 0] = 0
        return out + (s * x if s else 0)

    X64 = X.astype(np.float64)
    ref, scale = sums(X64), sums(np.abs(X64))
    with np.errstate(over="ignore"):
        fits = np.isfinite(ref.astype(np.float32))   # (two lowest values in a row, or 1.25 times one, do not)
    if op == "mean":
        deg = np.maximum(np.diff(rowptr), 1)[:, None]
        ref, scale = ref / deg, scale / deg
    got = Y.cpu().numpy()
    assert np.isneginf(got[~fits]).all() and np.isfinite(got[fits]).all()
    bad = fits & ~(np.abs(got - ref) <= TOL * scale + 1e-45)
    assert not bad.any(), [(int(r), int(c), float(X[r, c]), float(ref[r, c]), float(Y[r, c]), int(r % 3 + 1)) for r, c in np.argwhere(bad)[:5]]


@pytest.mark.parametrize("own", [1.0, 300.0, -1e5, LOWEST])
@pytest.mark.parametrize("k", [16, 50, 160])
def test_sets_that_do_not_hold_the_rows_own_column(env, k, own):
    """Node w is in a clique of its own and points at all of another one, of which only five nodes point back: that clique is a set of the row w without
    its column w, and what is in it counts though it is the only value there."""
    torch, cbm = env
    groups, big, small = 25, 20, 12
    n = groups * (big + small)
    nodes = np.random.default_rng(1).permutation(n).reshape(groups, big + small)
    src, dst = [], []
    for g in nodes:
        K, own_clique = g[:big], g[big:]
        w = own_clique[0]
        for c in (K, own_clique):
            src += [x for x in c for y in c if x != y]
            dst += [y for x in c for y in c if x != y]
        src += [w] * big + list(K[:5])
        dst += list(K) + [w] * 5
    order = np.lexsort((dst, src))
    src, dst = np.array(src)[order], np.array(dst, dtype=np.int32)[order]
    rowptr = np.concatenate(([0], np.cumsum(np.bincount(src, minlength=n)))).astype(np.int64)
    h = cbm.cbm_build(n, n, rowptr, dst)
    X = np.zeros((n, k), dtype=np.float32)
    ws = nodes[:, big]
    X[ws] = own                                            # beside nothing in its own clique, and one value (or none) in the other
    for c in range(k):
        if c % 3:
            X[nodes[:, c % big], c] = 3.0
    want = np.stack([X[dst[a:b]].astype(np.float64).sum(0) for a, b in zip(rowptr[:-1], rowptr[1:])])
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((n, k), float("nan"), device="cuda")
    assert _kinds(torch, cbm, h, lambda: cbm.cbm_spmm(h, Xd, Y)) == [6, 6]
    assert np.array_equal(Y.cpu().numpy()[ws], want[ws].astype(np.float32))
    cbm.cbm_spmm_mean(h, Xd, Y)
    assert np.allclose(Y.cpu().numpy()[ws], want[ws] / np.diff(rowptr)[ws, None], rtol=1e-6, atol=0)


def test_a_mask_on_a_graph_that_row_blocks_take_too(env, monkeypatch):
    """As the library chooses by itself: with shared sums and without, a row next to nothing but ordinary values is an ordinary value."""
    torch, cbm = env
    rowptr, colidx = _cliques(20000, twice=True)
    n, k = len(rowptr) - 1, 64
    X = torch.from_numpy(wl.gaussian_features(n, k, 2)).cuda()
    masked = torch.arange(0, n, 501, device="cuda")
    X[masked, 7] = LOWEST
    X[masked, 9] = -1e8
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    for sums, out, kinds in (("2", Y, [6, 6]), ("0", Z, [5])):
        monkeypatch.setenv("CBM_SHARED_SUMS", sums)
        monkeypatch.delenv("CBM_ROW_BLOCKS", raising=False)
        h = cbm.cbm_build(n, n, rowptr, colidx)
        assert _kinds(torch, cbm, h, lambda: cbm.cbm_spmm(h, X, out)) == kinds
    ok = Z.abs() < 1e6
    assert ok[masked].float().mean() > 0.9
    assert float((Y - Z).abs()[ok].max()) <= 1e-5 * 20 * 3


def test_streams_threads_and_captures_at_a_time(env, graph):
    """Products of one handle overlap freely: each stream and each capture has sums of its own, and what finds none does without, to the same bits."""
    torch, cbm = env
    g, k = graph, 64
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    Xs = [torch.from_numpy(wl.gaussian_features(g.n, k, s)).cuda() for s in range(24)]
    want = []
    for X in Xs:
        Y = torch.empty_like(X)
        cbm.cbm_spmm_normalized(h, X, Y)
        torch.cuda.synchronize()
        want.append(Y)
    # more streams than the handle has arrays for: the last ones sum each row's sets in place
    streams = [torch.cuda.Stream() for _ in Xs]
    Ys = [torch.full_like(X, float("nan")) for X in Xs]
    torch.cuda.synchronize()
    for _ in range(20):
        for s, X, Y in zip(streams, Xs, Ys):
            with torch.cuda.stream(s):
                cbm.cbm_spmm_normalized(h, X, Y)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(Ys, want))
    # host threads on one stream: the two launches of a product stay together
    errors = []

    def work(i):
        try:
            for _ in range(20):
                cbm.cbm_spmm_normalized(h, Xs[i], Ys[i])
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    for Y in Ys:
        Y.fill_(float("nan"))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors and all(torch.equal(a, b) for a, b in zip(Ys[:4], want))


def test_captured_products_replay_beside_others(env, graph):
    torch, cbm = env
    g, k = graph, 64
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    Xs = [torch.from_numpy(wl.gaussian_features(g.n, k, s)).cuda() for s in range(3)]
    Ys = [torch.empty_like(X) for X in Xs]
    graphs = []
    for X, Y in zip(Xs[:2], Ys[:2]):     # no product before the first capture
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            cbm.cbm_spmm_normalized(h, X, Y)
    side = [torch.cuda.Stream() for _ in range(2)]
    for it in range(4):
        for i, X in enumerate(Xs):
            X.copy_(torch.from_numpy(wl.gaussian_features(g.n, k, 10 + 3 * it + i)))
            Ys[i].fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(5):
            for s, gr in zip(side, graphs):
                with torch.cuda.stream(s):
                    gr.replay()
            cbm.cbm_spmm_normalized(h, Xs[2], Ys[2])
        torch.cuda.synchronize()
        for X, Y in zip(Xs, Ys):
            Z = torch.empty_like(X)
            cbm.cbm_spmm_normalized(h, X, Z)
            torch.cuda.synchronize()
            assert torch.equal(Y, Z)
    assert _err(Ys[0].cpu().numpy(), orc.spmm_csr_normalized(g.rowptr, g.colidx, Xs[0].cpu().numpy())) <= TOL


@pytest.fixture(scope="module")
def hubs(graph):
    """The graph with four nodes that have 700 neighbours more: rows of the paths that are split."""
    g = graph
    rng = np.random.default_rng(12)
    src = np.concatenate([np.repeat(np.arange(g.n), np.diff(g.rowptr)), np.repeat([5, 900, 1700, 2500], 700)])
    dst = np.concatenate([g.colidx.astype(np.int64), np.concatenate([rng.choice(g.n, 700, replace=False) for _ in range(4)])])
    return wl.graphs.csr_from_edges(g.n, src[src != dst], dst[src != dst])


@pytest.mark.parametrize("loops", [False, True])
@pytest.mark.parametrize("k", [7, 32, 64, 100, 300])
def test_products_without_memory_for_sums(env, hubs, k, loops):
    """More captures than the handle has arrays for, of a handle whose paths have split rows and share one scratch for them: all the same bits."""
    torch, cbm = env
    rowptr, colidx = hubs
    n = len(rowptr) - 1
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=loops)
    assert cbm.cbm_stats(h)["num_split_rows"] > 0
    Xs = [torch.from_numpy(wl.gaussian_features(n, k, s)).cuda() for s in range(20)]
    Xs[1][::7] *= 1e6                                # (rows that are put together without their own value)
    ops = [cbm.cbm_spmm, cbm.cbm_spmm_mean, lambda h, X, Y: cbm.cbm_spmm_gin(h, -1.0, X, Y)] + ([cbm.cbm_spmm_normalized, cbm.cbm_spmm_normalized_relu] if loops else [])
    Ys, graphs = [torch.empty_like(X) for X in Xs], []
    for i, (X, Y) in enumerate(zip(Xs, Ys)):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            ops[i % len(ops)](h, X, Y)
    streams = [torch.cuda.Stream() for _ in Xs]
    for _ in range(3):
        for Y in Ys:
            Y.fill_(float("nan"))
        torch.cuda.synchronize()
        for _ in range(4):
            for s, gr in zip(streams, graphs):
                with torch.cuda.stream(s):
                    gr.replay()
        torch.cuda.synchronize()
        for i, (X, Y) in enumerate(zip(Xs, Ys)):
            Z = torch.empty_like(X)
            assert _kinds(torch, cbm, h, lambda: ops[i % len(ops)](h, X, Z))[:2] == [6, 6]
            assert torch.equal(Y, Z), i
    ref = orc.spmm_csr(rowptr, colidx, Xs[0].cpu().numpy()) + (Xs[0].cpu().numpy().astype(np.float64) if loops else 0)
    assert _err(Ys[0].cpu().numpy(), ref) <= TOL


def test_streams_share_no_scratch_of_split_rows(env, hubs):
    torch, cbm = env
    rowptr, colidx = hubs
    n, k = len(rowptr) - 1, 96
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    Xs = [torch.from_numpy(wl.gaussian_features(n, k, s)).cuda() for s in range(24)]
    streams, Ys = [torch.cuda.Stream() for _ in Xs], [torch.full_like(X, float("nan")) for X in Xs]
    torch.cuda.synchronize()
    for _ in range(20):
        for s, X, Y in zip(streams, Xs, Ys):
            with torch.cuda.stream(s):
                cbm.cbm_spmm_normalized(h, X, Y)
    torch.cuda.synchronize()
    for X, Y in zip(Xs, Ys):
        assert _err(Y.cpu().numpy(), orc.spmm_csr_normalized(rowptr, colidx, X.cpu().numpy())) <= TOL


def _sixes(n):
    """Cliques of six."""
    members = np.random.default_rng(2).permutation(n).reshape(-1, 6)
    pairs = [(i, j) for i in range(6) for j in range(i)]
    return wl.graphs.csr_from_edges(n, np.concatenate([members[:, i] for i, _ in pairs]), np.concatenate([members[:, j] for _, j in pairs]))


def test_arrays_of_streams_and_graphs_that_are_done_come_back(env):
    """One stream after the other, one graph after the other: no more than a few arrays of 29 MiB, and every product has one.  Graphs that are not given
    up keep theirs, also beyond their own end."""
    torch, cbm = env
    n, k, array = 60000, 64, 29 << 20
    rowptr, colidx = _sixes(n)
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    X = torch.from_numpy(wl.integer_features(n, k, 1)).cuda()
    Y, want = torch.empty_like(X), torch.empty_like(X)
    cbm.cbm_spmm(h, X, want)
    torch.cuda.synchronize()

    def levels():
        cbm.cbm_profile_enable(h, True)
        cbm.cbm_spmm(h, X, Y)
        torch.cuda.synchronize()
        got = [r["level"] for r in cbm.cbm_profile_read(h)]
        cbm.cbm_profile_enable(h, False)
        return got

    free, streams = [], [torch.cuda.Stream() for _ in range(24)]
    for s in streams:
        with torch.cuda.stream(s):
            cbm.cbm_spmm(h, X, Y)
            s.synchronize()
            assert levels() == [1, 2]
        assert torch.equal(Y, want)
        free.append(torch.cuda.mem_get_info()[0])
    assert free[6] - free[-1] < array
    free, graphs = [], []
    for _ in range(24):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            cbm.cbm_spmm(h, X, Y)
        Y.fill_(float("nan"))
        for _ in range(3):
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
        del graph
        cbm.cbm_release_captures(h)
        free.append(torch.cuda.mem_get_info()[0])
    assert free[2] - free[-1] < array
    for _ in range(20):                       # more than there are arrays for, all alive: streams keep some
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            cbm.cbm_spmm(h, X, Y)
    for s in streams[:4]:
        with torch.cuda.stream(s):
            assert levels() == [1, 2]
    for graph in graphs:
        Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)
    with pytest.raises(cbm.CbmError):
        cbm.cbm_release_captures(cbm.cbm_build(n, n, rowptr, colidx, host_only=True))


def test_columns_in_goes(env, monkeypatch):
    """More sets than the arrays of sums have room for beside a wide X: the columns go through in several goes, the same sums."""
    torch, cbm = env
    n, k = 150000, 300
    members = np.random.default_rng(2).permutation(n).reshape(-1, 6)   # 25,000 cliques of six: 32 MiB hold 256 columns of sums
    src, dst = (np.concatenate([members[:, i] for i in range(6) for j in range(6) if i < j]), np.concatenate([members[:, j] for i in range(6) for j in range(6) if i < j]))
    rowptr, colidx = wl.graphs.csr_from_edges(n, src, dst)
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    X = torch.from_numpy(wl.integer_features(n, k, 1)).cuda()
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    assert _kinds(torch, cbm, h, lambda: cbm.cbm_spmm(h, X, Y)) == [6] * 4
    cbm.cbm_spmm_noalloc(h, X, Z)
    sums = torch.zeros(len(members), k, device="cuda").index_add_(0, torch.from_numpy(np.argsort(members.reshape(-1)) // 6).cuda(), X)
    want = sums[torch.from_numpy(np.argsort(members.reshape(-1)) // 6).cuda()]
    assert torch.equal(Y, want) and torch.equal(Z, want)


def test_nothing_is_allocated(env, graph):
    torch, cbm = env
    g = graph
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx)
    X = torch.from_numpy(wl.integer_features(g.n, 200, 1)).cuda()
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    cbm.cbm_spmm_noalloc(h, X[:, :8], Z[:, :8])  # (the kernels' code is on the GPU before memory is compared)
    cbm.cbm_spmm(h, X, Y)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    cbm.cbm_spmm_noalloc(h, X, Z)
    cbm.cbm_spmm(h, X, Y)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free and torch.equal(Y, Z)


@pytest.mark.parametrize("name,taken", [("collaboration", True), ("citation", False), ("rmat", False)])
def test_the_rule_takes_what_it_should(env, monkeypatch, name, taken):
    torch, cbm = env
    monkeypatch.delenv("CBM_SHARED_SUMS")
    g = wl.make_graph(name, **{"collaboration": dict(n=20000), "citation": dict(n=5000, p_in=1.6e-3, p_out=8e-5), "rmat": dict(scale=14)}[name])
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    X = torch.from_numpy(wl.gaussian_features(g.n, 64, 1)).cuda()
    Y = torch.empty_like(X)
    assert (6 in _kinds(torch, cbm, h, lambda: cbm.cbm_spmm_normalized(h, X, Y))) == taken
    assert _err(Y.cpu().numpy(), orc.spmm_csr_normalized(g.rowptr, g.colidx, X.cpu().numpy())) <= TOL
