"""Products in row blocks against the oracle: every epilogue, widths around the 32-column slab, strided and misaligned operands,
blocks that are not full, empty rows, directed graphs and their transpose, values that are not finite."""
import numpy as np
import pytest

import workloads as wl
from oracle import cbm_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 1e-5  # of a row's largest value, as for the paths: the products of the split are exact and the sums 32-bit ones


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2409_02208_amd as cbm

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch, cbm


@pytest.fixture(autouse=True)
def force(monkeypatch):
    monkeypatch.setenv("CBM_ROW_BLOCKS", "1")


def _err(got, ref, scale_from=None):
    d = np.abs(got.astype(np.float64) - ref).max(axis=1)
    s = np.abs(ref if scale_from is None else scale_from).max(axis=1)
    assert np.all(d[s == 0] == 0)
    return float((d[s > 0] / s[s > 0]).max()) if np.any(s > 0) else 0.0


def _in_blocks(torch, cbm, h, X, Y):
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, X, Y)
    torch.cuda.synchronize()
    kinds = [r["kind"] for r in cbm.cbm_profile_read(h)]
    cbm.cbm_profile_enable(h, False)
    return kinds == [5]


def _directed(n, seed):
    rng = np.random.default_rng(seed)
    rows = [np.unique(rng.integers(0, n, size=int(rng.integers(0, 40)))) if i % 7 else np.zeros(0, np.int64) for i in range(n)]
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    return rowptr, np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("n", [1, 33, 128, 129, 1000, 4099])
@pytest.mark.parametrize("k", [1, 31, 32, 33, 64, 100])
def test_sums_of_whole_numbers_are_exact(env, n, k):
    torch, cbm = env
    rowptr, colidx = _directed(n, n)
    h = cbm.cbm_build(n, n, rowptr, colidx)
    X = wl.integer_features(n, k, 3)
    Y = torch.full((n, k), float("nan"), device="cuda")
    Xd = torch.from_numpy(X).cuda()
    assert _in_blocks(torch, cbm, h, Xd, Y)
    ref = orc.spmm_csr(rowptr, colidx, X)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
    cbm.cbm_spmm_noalloc(h, Xd, Y.fill_(float("nan")))
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("layout", ["dense", "strided", "misaligned"])
@pytest.mark.parametrize("k", [16, 47, 128])
def test_every_epilogue(env, k, layout):
    torch, cbm = env
    g = wl.make_graph("protein", n=3000, knn=50)
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
    assert _err(run(cbm.cbm_spmm, h), plain) <= TOL


def test_directed_graph_and_its_transpose(env):
    torch, cbm = env
    n, k = 2000, 40
    rowptr, colidx = _directed(n, 9)
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    ht = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, transpose=True)
    X, G = (torch.from_numpy(wl.gaussian_features(n, k, s)).cuda() for s in (1, 2))
    Y, Z = torch.empty_like(X), torch.empty_like(X)
    cbm.cbm_spmm_normalized(h, X, Y)
    cbm.cbm_spmm_normalized(ht, G, Z)
    torch.cuda.synchronize()
    assert _err(Y.cpu().numpy(), orc.spmm_csr_normalized(rowptr, colidx, X.cpu().numpy())) <= TOL
    left, right = float((Y.double() * G.double()).sum()), float((X.double() * Z.double()).sum())
    assert abs(left - right) <= 1e-5 * float((Y.double() * G.double()).abs().sum())


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_values_that_are_not_finite_stay_in_their_rows(env, value):
    """A row whose columns hold no such value has the sum it has without it (the split multiplies by zero: 0 x inf)."""
    torch, cbm = env
    g = wl.make_graph("protein", n=1500, knn=30)
    k = 50
    X = wl.gaussian_features(g.n, k, 8)
    X[[3, 700], [0, 33]] = value
    with np.errstate(over="ignore", invalid="ignore"):
        A = np.zeros((g.n, g.n), dtype=bool)
        A[np.repeat(np.arange(g.n), np.diff(g.rowptr)), g.colidx] = True
        A[np.arange(g.n), np.arange(g.n)] = True
    touched = np.zeros((g.n, k), dtype=bool)
    touched[:, 0], touched[:, 33] = A[:, 3], A[:, 700]
    clean = X.copy()
    clean[[3, 700], [0, 33]] = 0.0
    hn = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    got = {}
    for name, x in (("with", X), ("without", clean)):
        Y = torch.empty((g.n, k), device="cuda")
        cbm.cbm_spmm_normalized(hn, torch.from_numpy(x).cuda(), Y)
        torch.cuda.synchronize()
        got[name] = Y.cpu().numpy()
    ref = orc.spmm_csr_normalized(g.rowptr, g.colidx, clean)
    assert _err(got["without"], ref) <= TOL
    untouched = np.abs(got["with"] - ref)[~touched] / np.broadcast_to(np.abs(ref).max(axis=1, keepdims=True), ref.shape)[~touched]
    assert untouched.max() <= TOL
    hit = got["with"][touched]
    if np.isfinite(value):
        assert np.isfinite(hit).all() and (hit > 1e36).all()
    else:
        assert np.isnan(hit).all() if np.isnan(value) else np.array_equal(hit, np.full_like(hit, value))


@pytest.mark.parametrize("form", ["rows", "hubs"])
@pytest.mark.parametrize("k", [33, 64])
def test_infinities_nan_and_large_values_beside_small_ones(env, monkeypatch, form, k):
    """Every sum is what its own entries make it: infinities of both signs, NaN, values that overflow only together or at 2^24 times
    their size, and in other rows of the same tile ordinary and the smallest values."""
    torch, cbm = env
    n = 1500
    if form == "rows":
        g = wl.make_graph("protein", n=n, knn=30)
        rowptr, colidx = g.rowptr, g.colidx
    else:
        for name, value in (("CBM_ROW_BLOCKS", "0"), ("CBM_HUB_BLOCKS", "2"), ("CBM_SPLIT_MIN", "128")):
            monkeypatch.setenv(name, value)
        rowptr, colidx = _popular(n, n, 4)
    rng = np.random.default_rng(k)
    X = wl.integer_features(n, k, 8).astype(np.float64)
    small = np.arange(0, k, 3)                       # columns of whole multiples of the smallest value, but for a few entries
    X[:, small] *= 2.0 ** -149
    where = rng.integers(0, n, 400), rng.integers(0, k, 400)
    X[where] = rng.choice([np.inf, -np.inf, np.nan, 3e38, -3e38, 2.0 ** 104, -(2.0 ** 100), 2.0 ** 90, 2.0 ** 87], 400)
    X = X.astype(np.float32)
    h = cbm.cbm_build(n, n, rowptr, colidx)
    Y = torch.empty((n, k), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
    got = Y.cpu().numpy()
    with np.errstate(all="ignore"):
        A = np.zeros((n, n))
        A[np.repeat(np.arange(n), np.diff(rowptr)), colidx] = 1.0
        finite = np.where(np.isfinite(X), X, 0.0).astype(np.float64)
        size = A @ np.abs(finite)
        ref = A @ finite
        up, down = A @ (np.isnan(X) | (X == np.inf)), A @ (np.isnan(X) | (X == -np.inf))
        over = np.abs(ref) >= 2.0 ** 128
        ref = np.where(up > 0, np.inf, np.where(over, np.sign(ref) * np.inf, ref))
        ref = np.where(down > 0, np.where(up > 0, np.nan, -np.inf), ref)
        near = np.abs(size) >= 2.0 ** 127   # may overflow on the way, or not
        same = np.isfinite(ref) & ~near
        assert np.array_equal(np.isnan(got)[~near], np.isnan(ref)[~near])
        assert np.array_equal(got[np.isinf(ref) & ~near], ref[np.isinf(ref) & ~near].astype(np.float32))
        assert np.all(np.abs(got - ref)[same] <= 2.0 ** -18 * size[same])
        exact = same & (size < 2.0 ** 24 * np.where(np.isin(np.arange(k), small), 2.0 ** -149, 1.0))
        assert exact.sum() > 0.3 * exact.size and np.array_equal(got[exact].astype(np.float64), ref[exact])


def test_values_that_are_not_finite_cost_little(env):
    """A tile summed again takes the matrix cores: about six times the product's time with NaN everywhere; a walk that selects entry by
    entry took sixteen times.  The line is at 11 to leave room for noise."""
    torch, cbm = env
    g = wl.make_graph("protein", n=20000, knn=150)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx)
    X, Y = torch.randn((g.n, 256), device="cuda"), torch.empty((g.n, 256), device="cuda")

    def best():
        times = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                cbm.cbm_spmm(h, X, Y)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    best()
    clean = best()
    X.fill_(float("nan"))
    assert best() <= 11 * clean
    X.normal_().mul_(1e-35)
    assert best() <= 2 * clean


@pytest.mark.parametrize("scale", [1e-36, 1e-34, 1e-30, 1e-27, 1e30])
def test_scale_of_the_values_does_not_matter(env, scale):
    torch, cbm = env
    g = wl.make_graph("protein", n=1500, knn=30)
    X = (wl.gaussian_features(g.n, 33, 8).astype(np.float64) * scale).astype(np.float32)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx)
    Y = torch.empty((g.n, 33), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
    torch.cuda.synchronize()
    assert _err(Y.cpu().numpy(), orc.spmm_csr(g.rowptr, g.colidx, X)) <= TOL


def test_handles_in_row_blocks_hold_and_count_the_blocks_only(env, monkeypatch):
    """The paths' arrays stay on the host, no scratch is sized for split rows that nothing launches, and bytes_cbm counts the blocks."""
    torch, cbm = env
    monkeypatch.setenv("CBM_SPLIT_MIN", "16")
    g = wl.make_graph("protein", n=6000, knn=80)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    stats = cbm.cbm_stats(h)
    assert stats["num_split_rows"] > 100
    X, Y = torch.ones((g.n, 32), device="cuda"), torch.empty((g.n, 32), device="cuda")
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm_normalized(h, X, Y)
    torch.cuda.synchronize()
    (r,) = cbm.cbm_profile_read(h)
    cbm.cbm_profile_enable(h, False)
    assert r["kind"] == 5
    # a block: its place and 128 rows; a column: its number and a bit for each of 128 rows
    assert stats["bytes_cbm"] == r["tasks"] * (12 + 4 * 128) + r["deltas"] * (4 + 16) + 4 * g.n
    free = torch.cuda.mem_get_info()[0]
    cbm.cbm_reserve(h, 65536)   # 100 split rows in 8 segments each would take 200 MB
    assert free - torch.cuda.mem_get_info()[0] < 16 << 20
    W = torch.eye(32, device="cuda")
    out, ws = torch.empty_like(Y), torch.empty(cbm.cbm_gcn2_workspace_bytes(h, 32, 32, 32), dtype=torch.uint8, device="cuda")
    cbm.cbm_gcn2_forward(h, X, W, W, out, ws)
    Xh = X.cpu().numpy()
    ref = orc.gcn2(g.rowptr, g.colidx, Xh, np.eye(32, dtype=np.float32), np.eye(32, dtype=np.float32))
    assert _err(out.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("form", ["rows", "hubs"])
def test_rows_of_x_beyond_32_bit_offsets(env, monkeypatch, form):
    """A leading dimension of 2^22: the kernel's large variant, which addresses X in 64 bits.  The last rows start beyond 4 GB."""
    torch, cbm = env
    n, k, ld = 700, 40, (1 << 22) + 4
    if form == "rows":
        rowptr, colidx = _directed(n, 9)
    else:
        for name, value in (("CBM_ROW_BLOCKS", "0"), ("CBM_HUB_BLOCKS", "2"), ("CBM_SPLIT_MIN", "128")):
            monkeypatch.setenv(name, value)
        rowptr, colidx = _popular(n, n, 4)
    h = cbm.cbm_build(n, n, rowptr, colidx)
    hn = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    room = torch.empty((n, ld), device="cuda")
    X, Y = room[:, 4:4 + k], torch.empty((n, k), device="cuda")
    Xi, Xg = wl.integer_features(n, k, 3), wl.gaussian_features(n, k, 5)
    X.copy_(torch.from_numpy(Xi))
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, X, Y)
    torch.cuda.synchronize()
    assert cbm.cbm_profile_read(h)[0]["kind"] == 5
    cbm.cbm_profile_enable(h, False)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, Xi))
    X.copy_(torch.from_numpy(Xg))
    norm, plain = orc.spmm_csr_normalized(rowptr, colidx, Xg), orc.spmm_csr(rowptr, colidx, Xg)
    for run, ref, scale in ((lambda: cbm.cbm_spmm_normalized(hn, X, Y), norm, None),
                            (lambda: cbm.cbm_spmm_normalized_relu(hn, X, Y), np.maximum(norm, 0), norm),
                            (lambda: cbm.cbm_spmm_mean(h, X, Y), orc.spmm_csr_mean(rowptr, colidx, Xg), None),
                            (lambda: cbm.cbm_spmm_gin(h, 0.5, X, Y), plain + 1.5 * Xg.astype(np.float64), None)):
        Y.fill_(float("nan"))
        run()
        assert _err(Y.cpu().numpy(), ref, scale) <= TOL


def test_more_columns_than_a_grid_has_slabs(env):
    """65,535 slabs of 32 columns and a few more: the gather kernels take them in one launch of 128 or 256 columns a block."""
    torch, cbm = env
    n, k = 5, 65535 * 32 + 37
    rowptr, colidx = np.array([0, 2, 2, 5, 6, 8]), np.array([0, 3, 1, 2, 4, 4, 0, 1], dtype=np.int32)
    X = torch.randint(-8, 9, (n, k), device="cuda").float()
    Y = torch.full((n, k), float("nan"), device="cuda")
    h = cbm.cbm_build(n, n, rowptr, colidx)
    cbm.cbm_spmm(h, X, Y)
    for i in range(n):
        assert torch.equal(Y[i], X[torch.from_numpy(colidx[rowptr[i]:rowptr[i + 1]]).cuda().long()].sum(0)), i
    cbm.cbm_spmm_gin(h, 1.0, X, Y)
    assert torch.equal(Y[0], X[0] + X[3] + 2 * X[0])


@pytest.mark.parametrize("unit", [2.0 ** -149, 2.0 ** -130, 2.0 ** -112])
def test_sums_of_the_smallest_values_are_exact(env, unit):
    """Whole multiples of the smallest 32-bit value (and of values whose lower parts are that small): nothing rounds, so every sum is
    exact, those of few small values and those that cancel to zero among them."""
    torch, cbm = env
    g = wl.make_graph("protein", n=1500, knn=30)
    X = wl.integer_features(g.n, 33, 8) * np.float64(unit)
    X[:, 5] = 0.0
    X[::50, 6] *= 4096.0 + 1.0
    X = X.astype(np.float32)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx)
    Y = torch.empty((g.n, 33), device="cuda")
    Xd = torch.from_numpy(X).cuda()
    assert _in_blocks(torch, cbm, h, Xd, Y)
    ref = orc.spmm_csr(g.rowptr, g.colidx, X)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref) and np.any(ref)


@pytest.mark.parametrize("scale", [1e-37, 1e-38, 1e-41])
def test_weights_take_no_value_below_what_the_parts_hold(env, scale):
    """x d^-1/2 is subnormal where x is not, or loses its last bits: the weighted sum over 300 columns is an ordinary value again."""
    torch, cbm = env
    g = wl.make_graph("protein", n=1500, knn=300)
    X = (np.abs(wl.gaussian_features(g.n, 33, 8)).astype(np.float64) * scale).astype(np.float32)
    h = cbm.cbm_build(g.n, g.n, g.rowptr, g.colidx, add_self_loops=True)
    Y = torch.empty((g.n, 33), device="cuda")
    cbm.cbm_spmm_normalized(h, torch.from_numpy(X).cuda(), Y)
    torch.cuda.synchronize()
    ref = orc.spmm_csr_normalized(g.rowptr, g.colidx, X)
    d = np.abs(Y.cpu().numpy().astype(np.float64) - ref)
    assert np.all(d <= 1e-6 * np.abs(ref) + 2.0 ** -149)  # (half a unit when the row weight makes a sum subnormal; w itself rounds by 2^-24)


# ---- hub blocks: the popular columns of the split rows of a matrix without a tree ----
def _popular(m, n, seed):
    """Rows of 150 to 700 entries among short ones, columns by a steep power law."""
    rng = np.random.default_rng(seed)
    rows = [np.unique((n * rng.random(int(rng.integers(150, 700)) if i % 3 == 0 else int(rng.integers(0, 20))) ** 3).astype(np.int64)) for i in range(m)]
    rowptr = np.zeros(m + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    return rowptr, np.concatenate(rows).astype(np.int32)


@pytest.fixture
def hubs(monkeypatch):
    monkeypatch.setenv("CBM_ROW_BLOCKS", "0")
    monkeypatch.setenv("CBM_HUB_BLOCKS", "2")
    monkeypatch.setenv("CBM_SPLIT_MIN", "128")


@pytest.mark.parametrize("m,n", [(700, 700), (1500, 900), (1000, 6000)])
@pytest.mark.parametrize("k", [1, 32, 47, 128])
def test_hub_blocks_sums_are_exact(env, hubs, m, n, k):
    torch, cbm = env
    rowptr, colidx = _popular(m, n, 4)
    h = cbm.cbm_build(m, n, rowptr, colidx)
    X = wl.integer_features(n, k, 3)
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((m, k), float("nan"), device="cuda")
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, Xd, Y)
    torch.cuda.synchronize()
    kinds = [r["kind"] for r in cbm.cbm_profile_read(h)]
    cbm.cbm_profile_enable(h, False)
    assert kinds[0] == 5 and 2 in kinds
    ref = orc.spmm_csr(rowptr, colidx, X)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
    cbm.cbm_spmm_noalloc(h, Xd, Y.fill_(float("nan")))
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), ref)
    cbm.cbm_spmm_mean(h, Xd, Y)
    assert _err(Y.cpu().numpy(), orc.spmm_csr_mean(rowptr, colidx, X)) <= TOL


@pytest.mark.parametrize("unit", [2.0 ** -149, 2.0 ** -130])
def test_hub_blocks_keep_the_smallest_values(env, hubs, unit):
    torch, cbm = env
    rowptr, colidx = _popular(700, 700, 4)
    X = (wl.integer_features(700, 40, 3) * np.float64(unit)).astype(np.float32)
    h = cbm.cbm_build(700, 700, rowptr, colidx)
    Y = torch.empty((700, 40), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(X).cuda(), Y)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, X))
    hn = cbm.cbm_build(700, 700, rowptr, colidx, add_self_loops=True)
    cbm.cbm_spmm_normalized(hn, torch.from_numpy(np.abs(X)).cuda(), Y)
    ref = orc.spmm_csr_normalized(rowptr, colidx, np.abs(X))
    # (a part of a row is rounded to the smallest value on its way through the scratch, as the gather kernels round theirs)
    assert np.all(np.abs(Y.cpu().numpy().astype(np.float64) - ref) <= 1e-6 * np.abs(ref) + 32 * 2.0 ** -149)


@pytest.mark.parametrize("k", [16, 47, 130])
def test_hub_blocks_normalised_and_transposed(env, hubs, k):
    torch, cbm = env
    n = 1200
    rowptr, colidx = _popular(n, n, 6)
    h = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True)
    ht = cbm.cbm_build(n, n, rowptr, colidx, add_self_loops=True, transpose=True)
    X, G = (torch.from_numpy(wl.gaussian_features(n, k, s)).cuda() for s in (1, 2))
    Y, Z, R = torch.empty_like(X), torch.empty_like(X), torch.empty_like(X)
    cbm.cbm_spmm_normalized(h, X, Y)
    cbm.cbm_spmm_normalized_relu(h, X, R)
    cbm.cbm_spmm_normalized(ht, G, Z)
    torch.cuda.synchronize()
    ref = orc.spmm_csr_normalized(rowptr, colidx, X.cpu().numpy())
    assert _err(Y.cpu().numpy(), ref) <= TOL
    assert _err(R.cpu().numpy(), np.maximum(ref, 0), ref) <= TOL
    left, right = float((Y.double() * G.double()).sum()), float((X.double() * Z.double()).sum())
    assert abs(left - right) <= 1e-5 * float((Y.double() * G.double()).abs().sum())
    cbm.cbm_spmm_gin(h, 0.5, X, Y)
    both = orc.spmm_csr(*_with_self(rowptr, colidx), X.cpu().numpy()) + 1.5 * X.cpu().numpy().astype(np.float64)
    assert _err(Y.cpu().numpy(), both) <= TOL


def test_hub_blocks_launch_records_count_work_items(env, hubs):
    """Scratch rows that the blocks write are no work items of the segment launch (its full-occupancy rule goes by them too)."""
    torch, cbm = env
    rowptr, colidx = _popular(1500, 1500, 4)
    h = cbm.cbm_build(1500, 1500, rowptr, colidx)
    X, Y = torch.ones((1500, 32), device="cuda"), torch.empty((1500, 32), device="cuda")
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, X, Y)
    torch.cuda.synchronize()
    records = cbm.cbm_profile_read(h)
    assert {1, 5} <= {r["kind"] for r in records}
    assert sum(r["tasks"] for r in records if r["kind"] in (0, 1)) == cbm.cbm_stats(h)["num_tasks"]


def _with_self(rowptr, colidx):
    rows = [np.union1d(colidx[rowptr[i]:rowptr[i + 1]], [i]) for i in range(len(rowptr) - 1)]
    rp = np.zeros(len(rowptr), dtype=np.int64)
    rp[1:] = np.cumsum([len(r) for r in rows])
    return rp, np.concatenate(rows).astype(np.int32)


def test_hub_blocks_take_noalloc_columns_in_goes(env, hubs, monkeypatch):
    """Hub blocks can need more scratch than the limit goes by (that of the handle without them): the columns then come in
    goes; what was refused is refused.  Pieces of one group make the scratch large: 64 MiB at about 58 columns, where the limit
    lies at about 524."""
    torch, cbm = env
    monkeypatch.setenv("CBM_HUB_PIECE", "1")
    monkeypatch.setenv("CBM_REST_WHOLE", "0")
    m, n = 12000, 12000
    rowptr, colidx = _popular(m, n, 5)
    h = cbm.cbm_build(m, n, rowptr, colidx)
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, torch.zeros((n, 4), device="cuda"), torch.empty((m, 4), device="cuda"))
    torch.cuda.synchronize()
    tasks = {r["kind"]: r["tasks"] for r in cbm.cbm_profile_read(h)}
    cbm.cbm_profile_enable(h, False)
    # a scratch row for each segment and for each of a piece's rows (the last block of 128 may be short, and has the fewest pieces)
    slots = tasks[1] + 128 * (tasks[5] - tasks[5] // (4000 // 128))
    assert slots * 128 > 16 << 20, "widths from 128 on take several goes"
    monkeypatch.setenv("CBM_HUB_BLOCKS", "0")
    plain = cbm.cbm_build(m, n, rowptr, colidx)
    refused = []
    for k in range(64, 1600, 64):
        X = torch.randint(-3, 4, (n, k), device="cuda").float()
        Y, Z = torch.empty((m, k), device="cuda"), torch.empty((m, k), device="cuda")
        got = []
        for handle, out in ((h, Y), (plain, Z)):
            try:
                cbm.cbm_spmm_noalloc(handle, X, out)
                got.append(True)
            except cbm.CbmError as e:
                assert e.status == 5
                got.append(False)
        assert got[0] == got[1], k
        if not got[0]:
            refused.append(k)
            break
        torch.cuda.synchronize()
        assert torch.equal(Y, Z), k
    assert k > 448, "widths with several goes were to be tried"
    assert refused, "widths up to the limit were to be tried"


# ---- column-blocked handles: the blocks are those of the inner handle, whose rows are parts of rows ----
def _kinds(torch, cbm, h, n, k):
    cbm.cbm_profile_enable(h, True)
    cbm.cbm_spmm(h, torch.ones((n, k), device="cuda"), torch.empty((cbm.cbm_stats(h)["m"], k), device="cuda"))
    torch.cuda.synchronize()
    kinds = {r["kind"] for r in cbm.cbm_profile_read(h)}
    cbm.cbm_profile_enable(h, False)
    return kinds


@pytest.mark.parametrize("k", [32, 47])
def test_column_blocked_handle_with_hub_blocks_inside(env, hubs, k):
    torch, cbm = env
    n = 1200
    rowptr, colidx = _popular(n, n, 6)
    h = cbm.cbm_build(n, n, rowptr, colidx, column_blocks=2)
    hn = cbm.cbm_build(n, n, rowptr, colidx, column_blocks=2, add_self_loops=True)
    assert {4, 5} <= _kinds(torch, cbm, h, n, k) and {4, 5} <= _kinds(torch, cbm, hn, n, k)
    Xi, Xg = wl.integer_features(n, k, 3), wl.gaussian_features(n, k, 5)
    Y = torch.full((n, k), float("nan"), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(Xi).cuda(), Y)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, Xi))
    X = torch.from_numpy(Xg).cuda()
    norm, plain = orc.spmm_csr_normalized(rowptr, colidx, Xg), orc.spmm_csr(rowptr, colidx, Xg)
    for run, ref, scale in ((lambda: cbm.cbm_spmm_normalized(hn, X, Y), norm, None),
                            (lambda: cbm.cbm_spmm_normalized_relu(hn, X, Y), np.maximum(norm, 0), norm),
                            (lambda: cbm.cbm_spmm_mean(h, X, Y), orc.spmm_csr_mean(rowptr, colidx, Xg), None),
                            (lambda: cbm.cbm_spmm_gin(h, 0.5, X, Y), plain + 1.5 * Xg.astype(np.float64), None)):
        Y.fill_(float("nan"))
        run()
        assert _err(Y.cpu().numpy(), ref, scale) <= TOL


@pytest.mark.parametrize("k", [32, 47])
def test_column_blocked_handle_with_row_blocks_inside(env, k):
    """Two part-rows a row and twice as many columns as rows: the inner matrix is square and takes row blocks."""
    torch, cbm = env
    m, n = 700, 1400
    rng = np.random.default_rng(4)
    rows = [np.unique(rng.integers(0, n, size=int(rng.integers(0, 40)))) for _ in range(m)]
    rowptr = np.zeros(m + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    colidx = np.concatenate(rows).astype(np.int32)
    h = cbm.cbm_build(m, n, rowptr, colidx, column_blocks=2)
    assert _kinds(torch, cbm, h, n, k) == {4, 5}
    Xi, Xg = wl.integer_features(n, k, 3), wl.gaussian_features(n, k, 5)
    Y = torch.full((m, k), float("nan"), device="cuda")
    cbm.cbm_spmm(h, torch.from_numpy(Xi).cuda(), Y)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), orc.spmm_csr(rowptr, colidx, Xi))
    cbm.cbm_spmm_mean(h, torch.from_numpy(Xg).cuda(), Y)
    assert _err(Y.cpu().numpy(), orc.spmm_csr_mean(rowptr, colidx, Xg)) <= TOL
