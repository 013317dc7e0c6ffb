"""Dense matmul through bf16 parts (every kernel of it, forced) and the panel kernel on a B of any alignment."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_2409_02208_amd as cbm

    assert torch.cuda.is_available(), "these tests need the MI355X"
    return torch, cbm


def _product(env, A, B, pad=(0, 0, 0)):
    torch, cbm = env
    bufs = []
    for x, p in ((A, pad[0]), (B, pad[1])):
        t = torch.zeros((x.shape[0], x.shape[1] + p), device="cuda")[:, p // 2:p // 2 + x.shape[1]]
        t.copy_(torch.from_numpy(x))
        bufs.append(t)
    room = torch.full((A.shape[0], B.shape[1] + pad[2]), float("nan"), device="cuda")
    C = room[:, pad[2] // 2:pad[2] // 2 + B.shape[1]]
    cbm.cbm_dense_matmul(bufs[0], bufs[1], C)
    torch.cuda.synchronize()
    got = room.cpu().numpy()
    outside = np.delete(got, np.arange(pad[2] // 2, pad[2] // 2 + B.shape[1]), axis=1)
    assert np.isnan(outside).all(), "wrote outside the columns"
    return got[:, pad[2] // 2:pad[2] // 2 + B.shape[1]]


WIDTHS = {1: (1, 16, 31, 32), 2: (33, 47, 64), 3: (65, 128, 130), 4: (65, 128, 250)}


@pytest.mark.parametrize("form", [1, 2, 3, 4])
@pytest.mark.parametrize("m,k", [(1, 1), (31, 17), (33, 16), (127, 32), (129, 33), (300, 100), (257, 500)])
def test_every_kernel_within_the_componentwise_bound(env, monkeypatch, form, m, k):
    monkeypatch.setenv("CBM_GEMM_SPLIT", str(form))
    rng = np.random.default_rng(form * 1000 + m + k)
    for n in WIDTHS[form]:
        for pad in ((0, 0, 0), (3, 5, 1)):
            A, B = (rng.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n)))
            got = _product(env, A, B, pad)
            ref = A.astype(np.float64) @ B.astype(np.float64)
            # a rounding of at most 2^-24 for each of K additions, of the waves' shares, and of the small sums at the end; the
            # products of parts that are left out are below 1.01 * 2^-24 of a term
            bound = (k + 6) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))
            assert np.all(np.abs(got - ref) <= bound + 1e-37), (n, pad)
            Ai, Bi = (rng.integers(-9, 10, s).astype(np.float32) for s in ((m, k), (k, n)))
            assert np.array_equal(_product(env, Ai, Bi, pad).astype(np.float64), Ai.astype(np.float64) @ Bi.astype(np.float64))


@pytest.mark.parametrize("form", [1, 2, 3, 4])
@pytest.mark.parametrize("k", [1, 2, 5, 16, 17, 32])
def test_worst_mantissas_lose_no_more_than_a_rounding(env, monkeypatch, form, k):
    """Mantissas whose lower parts are as large as they get, all of one sign: what is left out would add up.  The products left out
    are below 1.01 * 2^-24 of a term; a step of 16 rounds the large sum once (at most two steps here), the small sums are
    added once, and their own roundings are 2^-8 of that."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", str(form))
    bits = np.array([0x3F80FFFF, 0x3F807FFF, 0x3F808001, 0x3F8080FF, 0x3F80FF80, 0x3FFF7FFF, 0x3F817F7F, 0x3F80FFFE], dtype=np.uint32)
    v = bits.view(np.float32)
    rng = np.random.default_rng(k)
    for n in WIDTHS[form]:
        A, B = v[rng.integers(0, len(v), (70, k))], v[rng.integers(0, len(v), (k, n))]
        A[0], B[:, 0] = v[0], v[0]
        got = _product(env, A, B)
        ref = A.astype(np.float64) @ B.astype(np.float64)
        assert (np.abs(got - ref) / ref).max() <= ((k + 15) // 16 + 2.1) * 2.0 ** -24, n


@pytest.mark.parametrize("form", [1, 2, 3, 4])
@pytest.mark.parametrize("k,nonzeros", [(128, 1), (500, 4), (500, 10), (500, 50), (96, 96), (500, 500)])
def test_error_is_no_larger_than_that_of_the_fp32_kernels(env, monkeypatch, form, k, nonzeros):
    """Dense rows, and sparse ones, where no long chain of additions hides what a product loses.  (One term a row: 2 to 3 % more than
    one rounding, because of the products left out; measured 2.60e-8 against 2.53e-8.)"""
    rng = np.random.default_rng(k + nonzeros)
    m, n = 2000, WIDTHS[form][-1]
    for positive in (False, True):
        A, B = np.zeros((m, k), np.float32), rng.standard_normal((k, n), dtype=np.float32)
        at = rng.random((m, k)).argsort(axis=1)[:, :nonzeros]
        np.put_along_axis(A, at, rng.standard_normal((m, nonzeros), dtype=np.float32), axis=1)
        if positive:
            A, B = np.abs(A), np.abs(B)
        ref = A.astype(np.float64) @ B.astype(np.float64)
        err = {}
        for which in ("0", str(form)):
            monkeypatch.setenv("CBM_GEMM_SPLIT", which)
            err[which] = np.linalg.norm(_product(env, A, B) - ref) / np.linalg.norm(ref)
        assert err[str(form)] <= (1.05 if nonzeros == 1 else 1.0) * err["0"], err


@pytest.mark.parametrize("form", [1, 2, 3, 4])
def test_values_that_have_no_parts(env, monkeypatch, form):
    """Infinities and NaN reach the outputs they reach by definition and no others; very small operands keep their precision."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", str(form))
    rng = np.random.default_rng(form)
    m, k, n = 200, 70, WIDTHS[form][-1]
    A, B = (rng.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n)))
    A[7, 3], A[100, 5], B[9, 11] = np.inf, np.nan, -np.inf
    got = _product(env, A, B)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    ok = np.isfinite(ref)
    assert np.abs(got - ref)[ok].max() <= 1e-4
    for a, b in ((1e-36, 1.0), (1e-35, 1e10), (1.0, 1e-36), (1e30, 1.0)):
        A, B = (rng.standard_normal(s).astype(np.float64) for s in ((m, k), (k, n)))
        A, B = (A * a).astype(np.float32), (B * b).astype(np.float32)
        ref = A.astype(np.float64) @ B.astype(np.float64)
        assert np.linalg.norm(_product(env, A, B) - ref) <= 1e-6 * np.linalg.norm(ref), (a, b)


@pytest.mark.parametrize("form", [1, 2, 3, 4])
@pytest.mark.parametrize("a,b", [(1e-41, 1e37), (1e-41, 1e30), (1e-39, 1e10), (1e-39, 1.0), (1e10, 1e-40), (1e-22, 1e-22), (2.0 ** -149, 1.0)])
def test_values_too_small_for_the_parts_are_not_lost(env, monkeypatch, form, a, b):
    """Operands that are subnormal or nearly so, all of them or some: no sum may vanish.  A result keeps K roundings, and half of the
    smallest fp32 value where it is subnormal itself."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", str(form))
    rng = np.random.default_rng(form)
    m, k, n = 70, 40, WIDTHS[form][-1]
    A = (rng.integers(1, 9, (m, k)) * np.float64(a)).astype(np.float32)
    B = (rng.integers(1, 9, (k, n)) * np.float64(b)).astype(np.float32)
    A[3], B[:, 1] = 0.0, 0.0
    A[5, 7:] = 0.0                      # one small value among zeros
    ref = A.astype(np.float64) @ B.astype(np.float64)
    got = _product(env, A, B)
    assert np.all(np.abs(got - ref) <= (k + 6) * 2.0 ** -24 * np.abs(ref) + 2.0 ** -149)
    assert np.all(got[3] == 0) and np.all(got[:, 1] == 0)
    A[:, ::2] *= -1.0                   # either sign, beside ordinary rows
    A[9] = 1e-3
    ref, size = A.astype(np.float64) @ B.astype(np.float64), np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    assert np.all(np.abs(_product(env, A, B) - ref) <= (k + 6) * 2.0 ** -24 * size + 2.0 ** -149)


@pytest.mark.parametrize("value", ["6", "-1", "17", "2x", "", "yes"])
def test_the_switch_takes_no_other_value(env, monkeypatch, value):
    rng = np.random.default_rng(3)
    A, B = rng.standard_normal((300, 30), dtype=np.float32), rng.standard_normal((30, 33), dtype=np.float32)  # the fp32 kernels' by the rule
    monkeypatch.delenv("CBM_GEMM_SPLIT", raising=False)
    want = _product(env, A, B)
    monkeypatch.setenv("CBM_GEMM_SPLIT", value)
    assert np.array_equal(_product(env, A, B), want)
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    assert np.array_equal(_product(env, A, B), want)
    for kernel in ("2", "5"):
        monkeypatch.setenv("CBM_GEMM_SPLIT", kernel)
        assert not np.array_equal(_product(env, A, B), want)


@pytest.mark.parametrize("k,n", [(500, 64), (500, 7), (256, 256), (300, 96)])
def test_values_that_are_not_finite_cost_little(env, k, n):
    """Tiles computed again take the fp32 matrix cores: at most four times the product's time with NaN everywhere (measured), not the
    40 to 120 times of a chain per element; the line is at 12 to leave room for noise."""
    torch, cbm = env
    A, B, C = torch.randn(20000, k, device="cuda"), torch.randn(k, n, device="cuda"), torch.empty(20000, n, device="cuda")

    def best():
        us = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                cbm.cbm_dense_matmul(A, B, C)
            b.record()
            torch.cuda.synchronize()
            us.append(a.elapsed_time(b))
        return min(us)

    best()
    clean = best()
    B[3, 2] = float("inf")
    assert best() <= 12 * clean
    A.fill_(float("nan"))
    assert best() <= 12 * clean


# just tall enough for the panel kernel; and just deep or tall enough for it to take a B of any width
@pytest.mark.parametrize("m,k,n", [(8193, 36, n) for n in (16, 17, 47, 112, 130)] +
                         [(8193, 48, 65), (8193, 48, 130), (32769, 256, 47), (49153, 100, 33), (131073, 48, 17)])
def test_panel_kernel_on_any_b(env, monkeypatch, m, k, n):
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    rng = np.random.default_rng(n)
    A, B = (rng.integers(-9, 10, s).astype(np.float32) for s in ((m, k), (k, n)))
    ref = A.astype(np.float64) @ B.astype(np.float64)
    for pad in ((0, 0, 0), (4, 1, 3), (4, 3, 0)):
        A4 = (pad[0] // 4 * 4, pad[1], pad[2])
        torch, cbm = env
        Ad = torch.zeros((m, k + A4[0]), device="cuda")[:, :k]
        Ad.copy_(torch.from_numpy(A))
        Bd = torch.zeros((k, n + A4[1]), device="cuda")[:, A4[1] // 2:A4[1] // 2 + n]
        Bd.copy_(torch.from_numpy(B))
        C = torch.full((m, n + A4[2]), float("nan"), device="cuda")[:, :n]
        cbm.cbm_dense_matmul(Ad, Bd, C)
        torch.cuda.synchronize()
        assert np.array_equal(C.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("k", [4, 16, 32, 36, 48, 64, 68, 80, 84, 96, 100, 112, 116, 128, 132, 144, 160, 176, 200, 240, 320])
@pytest.mark.parametrize("n", [16, 32, 48, 64, 112])
def test_depths_of_the_panel_kernel(env, monkeypatch, k, n):
    """K of every remainder of the groups that a wave keeps in flight, with fewer groups of rows than waves: whole numbers, bit for bit."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    torch, cbm = env
    gen = torch.Generator(device="cuda").manual_seed(k * 1000 + n)
    for m in (8192, 8209):
        A = torch.randint(-8, 9, (m, k), device="cuda", generator=gen).float()
        B = torch.randint(-8, 9, (k, n), device="cuda", generator=gen).float()
        C = torch.full((m, n), float("nan"), device="cuda")
        cbm.cbm_dense_matmul(A, B, C)
        assert torch.equal(C.double(), A.double() @ B.double()), (m, k, n)


@pytest.mark.parametrize("k", [48, 64, 80, 100, 112, 144, 160, 224])
@pytest.mark.parametrize("n", [16, 32, 48, 64])
def test_depths_of_the_panel_kernel_with_whole_groups(env, monkeypatch, k, n):
    """Rows beyond 32 for each of its 2,048 waves, one group after the other in a wave and the next one's rows asked for by the last pass of the one before; what is
    left over goes out in single column tiles, in pairs of them and whole (left over here: 1,000 and 1,500 groups of nothing else, then 2, 1,000, 1,500 and 1)."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    torch, cbm = env
    gen = torch.Generator(device="cuda").manual_seed(k * 1000 + n)
    for m in (31995, 47995, 65569, 97531, 113531, 131077):
        A = torch.randint(-8, 9, (m, k), device="cuda", generator=gen).float()
        B = torch.randint(-8, 9, (k, n), device="cuda", generator=gen).float()
        C = torch.full((m, n), float("nan"), device="cuda")
        cbm.cbm_dense_matmul(A, B, C)
        assert torch.equal(C.double(), A.double() @ B.double()), (m, k, n)


@pytest.mark.parametrize("k", [764, 768, 772, 784, 788, 1088, 1092, 1104, 1120, 1124])
@pytest.mark.parametrize("n", [17, 24, 31, 32, 33, 40, 47, 48])
def test_deepest_panels(env, monkeypatch, k, n):
    """On both sides of where the panel fits: B of even widths and of odd ones end at different depths."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    torch, cbm = env
    gen = torch.Generator(device="cuda").manual_seed(k * 1000 + n)
    for m in (8192, 66000):
        A = torch.randint(-8, 9, (m, k), device="cuda", generator=gen).float()
        B = torch.randint(-8, 9, (k, n), device="cuda", generator=gen).float()
        C = torch.full((m, n), float("nan"), device="cuda")
        cbm.cbm_dense_matmul(A, B, C)
        assert torch.equal(C.double(), A.double() @ B.double()), (m, k, n)
