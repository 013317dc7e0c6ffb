"""Dense matmul with B held in registers: every width, number of steps and number of waves that share K, at their edges."""
import numpy as np
import pytest

import test_gpu_matmul_split as split
from test_gpu_matmul_split import _product, env  # noqa: F401

pytestmark = pytest.mark.gpu
WIDTHS = (1, 16, 17, 32, 33, 48, 49, 64)


# K on both sides of every step of 32 and of what one, four and eight waves hold, for rows enough for all waves or not
@pytest.mark.parametrize("k", [1, 3, 8, 31, 32, 33, 64, 65, 96, 97, 100, 128, 129, 200, 256, 257, 301, 320, 384, 385, 500, 512, 513, 768, 769, 1000, 1024, 1025])
def test_whole_numbers_come_out_exactly(env, monkeypatch, k):  # noqa: F811
    monkeypatch.setenv("CBM_GEMM_SPLIT", "5")
    torch, cbm = env
    gen = torch.Generator(device="cuda").manual_seed(k)
    for n in WIDTHS:
        for m in (1, 15, 17, 8192, 8200) + ((17001, 33333, 51001) if n in (16, 48, 64) else ()):  # (from 32,768 on waves have several tiles of rows)
            for pad in ((0, 0, 0), (4, 0, 1), (3, 1, 0)):
                A, B = (torch.randint(-9, 10, s, device="cuda", generator=gen).float() for s in ((m, k + pad[0]), (k, n + pad[1])))
                A, B, C = A[:, pad[0] // 2:][:, :k], B[:, :n], torch.full((m, n + pad[2]), float("nan"), device="cuda")
                cbm.cbm_dense_matmul(A, B, C[:, :n])
                assert torch.equal(C[:, :n].double(), A.double() @ B.double()), (m, n, pad)
                assert bool(C[:, n:].isnan().all()), "wrote outside the columns"


# two, three and four panels of columns, the last of them narrow or not; by the rule, on both sides of its lines, and whatever it says
@pytest.mark.parametrize("n", [65, 80, 81, 96, 97, 112, 128, 129, 160, 193, 255, 256, 257])
def test_panels_of_columns(env, monkeypatch, n):  # noqa: F811
    torch, cbm = env
    gen = torch.Generator(device="cuda").manual_seed(n)
    for m, k in ((17, 9), (2048, 65), (2049, 65), (4097, 40), (32768, 64), (32767, 33), (65537, 100), (9000, 300), (40000, 32), (3, 800)):
        A, B = (torch.randint(-9, 10, s, device="cuda", generator=gen).float() for s in ((m, k), (k, n + 3)))
        for form in (None, "5"):
            monkeypatch.delenv("CBM_GEMM_SPLIT", raising=False) if form is None else monkeypatch.setenv("CBM_GEMM_SPLIT", form)
            C = torch.full((m, n + 1), float("nan"), device="cuda")
            cbm.cbm_dense_matmul(A, B[:, 1:n + 1], C[:, :n])
            assert torch.equal(C[:, :n].double(), A.double() @ B[:, 1:n + 1].double()), (m, k, form)
            assert bool(C[:, n:].isnan().all()), "wrote outside the columns"


@pytest.mark.parametrize("m,k", [(1, 1), (31, 17), (129, 33), (300, 100), (257, 500), (9000, 300)])
def test_within_the_componentwise_bound(env, monkeypatch, m, k):  # noqa: F811
    monkeypatch.setenv("CBM_GEMM_SPLIT", "5")
    rng = np.random.default_rng(m + k)
    for n in WIDTHS:
        A, B = (rng.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n)))
        ref = A.astype(np.float64) @ B.astype(np.float64)
        # a rounding of at most 2^-24 for each of K additions, and of the small sums at the end
        bound = (k + 6) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))
        assert np.all(np.abs(_product(env, A, B) - ref) <= bound + 1e-37), n


@pytest.mark.parametrize("m", [2000, 10000])
@pytest.mark.parametrize("k,n", [(8, 16), (32, 64), (100, 47), (128, 64), (200, 33), (320, 64), (500, 64), (500, 7), (768, 40), (32, 200), (100, 80), (256, 112)])
def test_error_is_no_larger_than_that_of_the_kernels_before(env, monkeypatch, m, k, n):  # noqa: F811
    """The fp32 kernels, and the kernel of parts for short and deep products (at m = 2000: 640,000 roundings in each 2-norm for n = 64, 3 % is noise)."""
    rng = np.random.default_rng(k + n)
    A, B = (rng.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n)))
    ref = A.astype(np.float64) @ B.astype(np.float64)
    err = {}
    for which in ("0", "2" if n <= 64 else "4", "5"):
        monkeypatch.setenv("CBM_GEMM_SPLIT", which)
        err[which] = np.linalg.norm(_product(env, A, B) - ref) / np.linalg.norm(ref)
    assert err["5"] <= err["0"] and err["5"] <= 1.03 * min(err.values()), err


@pytest.fixture
def widths(monkeypatch):
    monkeypatch.setitem(split.WIDTHS, 5, (16, 33, 64))


@pytest.mark.parametrize("k", [1, 2, 5, 16, 17, 32])
def test_worst_mantissas_lose_no_more_than_a_rounding(env, monkeypatch, widths, k):  # noqa: F811
    split.test_worst_mantissas_lose_no_more_than_a_rounding(env, monkeypatch, 5, k)


def test_values_that_have_no_parts(env, monkeypatch, widths):  # noqa: F811
    split.test_values_that_have_no_parts(env, monkeypatch, 5)


@pytest.mark.parametrize("a,b", [(1e-41, 1e37), (1e-39, 1.0), (1e10, 1e-40), (1e-22, 1e-22), (2.0 ** -149, 1.0)])
def test_values_too_small_for_the_parts_are_not_lost(env, monkeypatch, widths, a, b):  # noqa: F811
    split.test_values_too_small_for_the_parts_are_not_lost(env, monkeypatch, 5, a, b)


@pytest.mark.parametrize("k", [20, 200, 600])
def test_values_that_are_not_finite(env, monkeypatch, k):  # noqa: F811
    """They reach the outputs they reach by definition, where K is one wave's, four waves' and eight's; beyond K and N nothing is read as a value."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", "5")
    rng = np.random.default_rng(k)
    for n in (7, 33, 64):
        for m in (40, 9000):
            A, B = (rng.standard_normal(s, dtype=np.float32) for s in ((m, k), (k, n)))
            A[7, 3], A[30, k - 1], B[k // 2, n - 2], A[m - 1, 0] = np.inf, np.nan, -np.inf, 3e37  # (times 5, more than |B| gets to: finite)
            with np.errstate(invalid="ignore"):
                ref = A.astype(np.float64) @ B.astype(np.float64)
            got = _product(env, A, B, (2, 1, 0))
            with np.errstate(over="ignore"):
                ref32 = ref.astype(np.float32)
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref32)], ref32[np.isinf(ref32)])
            ok = np.isfinite(ref32)
            size = np.abs(np.nan_to_num(A, posinf=0, neginf=0)).astype(np.float64) @ np.abs(np.nan_to_num(B, posinf=0, neginf=0)).astype(np.float64)
            assert np.all(np.abs(got - ref)[ok] <= (k + 6) * 2.0 ** -24 * size[ok])


# one wave, two, four and eight, for few rows and many; panels of columns beside it
@pytest.mark.parametrize("m", [2000, 20000])
@pytest.mark.parametrize("k,n", [(20, 32), (128, 47), (150, 16), (300, 64), (500, 64), (700, 33), (32, 200), (256, 96)])
def test_a_row_of_one_term_is_rounded_once(env, monkeypatch, m, k, n):  # noqa: F811
    """As the fp32 kernels do it.  Left out is the product of the lowest parts, at most 2^-34 of the term; the small products are below 2^-6.9 of it and are added in
    seven roundings: together below 2^-28, beside the one rounding of 2^-24 at the end."""
    rng = np.random.default_rng(k + n)
    A, B = np.zeros((m, k), np.float32), rng.standard_normal((k, n), dtype=np.float32)
    A[np.arange(m), rng.integers(0, k, m)] = rng.standard_normal(m, dtype=np.float32)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    err = {}
    for which in ("0", "5"):
        monkeypatch.setenv("CBM_GEMM_SPLIT", which)
        got = _product(env, A, B)
        assert np.all(np.abs(got - ref) <= (1 + 2.0 ** -4) * 2.0 ** -24 * np.abs(ref) + 2.0 ** -150), which
        err[which] = np.linalg.norm(got - ref)
    assert err["5"] <= (1 + 2.0 ** -10) * err["0"], err


@pytest.mark.parametrize("k,nonzeros", [(128, 1), (500, 4), (500, 10), (500, 50), (96, 96), (500, 500)])
def test_error_is_no_larger_than_that_of_the_fp32_kernels(env, monkeypatch, widths, k, nonzeros):  # noqa: F811
    split.test_error_is_no_larger_than_that_of_the_fp32_kernels(env, monkeypatch, 5, k, nonzeros)


# waves that share K or not, with several tiles of 16 rows one after the other; three tiles of columns, and two panels of them
@pytest.mark.parametrize("k", [30, 100, 190, 300, 500, 760])
@pytest.mark.parametrize("n", [5, 47, 96])
def test_sums_that_are_not_finite_among_others(env, monkeypatch, k, n):  # noqa: F811
    """Whole numbers with infinities, NaN and values from 2^104 on in a single row, in rows of tiles that follow each other in a workgroup, in the first rows and the
    last: these reach what they reach by definition, and all other sums come out exactly."""
    monkeypatch.setenv("CBM_GEMM_SPLIT", "5")
    rng = np.random.default_rng(k + n)
    m = 20011
    A, B = (rng.integers(-9, 10, s).astype(np.float32) for s in ((m, k), (k, n)))
    rows = np.unique(np.concatenate(([0, m - 1, m - 12], rng.integers(0, m, 60), np.arange(4096, 4096 + 16 * 300, 16))))  # (one each: two would cancel)
    A[rows, rng.integers(0, k, len(rows))] = rng.choice(np.float32([np.inf, -np.inf, np.nan, 2.0 ** 104, -2.0 ** 110]), len(rows))
    for column in (None, n - 1):
        if column is not None:
            B[k // 3, column] = np.inf
        with np.errstate(invalid="ignore"):
            ref = A.astype(np.float64) @ B.astype(np.float64)
        got = _product(env, A, B, (1, 0, 1)).astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        small = np.abs(ref) < 2.0 ** 24
        assert np.array_equal(got[small], ref[small])
        large = np.isfinite(ref) & ~small  # one value of 2^104 or more decides
        assert np.all(np.abs(got - ref)[large] <= 2.0 ** -23 * np.abs(ref[large]))


# products of the fp32 kernels, and of the kernels of parts in each of their forms: there without the products ml and lm, as they do it
@pytest.mark.parametrize("m,k,n,otherwise", [(24577, 128, 16, "0"), (24576, 128, 16, "1"), (8193, 300, 7, "1"), (20000, 500, 64, "2"), (24576, 700, 33, "2"), (24577, 500, 64, "0"),
                                             (4000, 32, 65, "3"), (4000, 31, 65, "0"), (36000, 192, 112, "3"), (2000, 500, 200, "3"), (66000, 256, 128, "4"), (66000, 95, 128, "0")])
def test_as_near_to_64_bits_as_what_would_run_otherwise(env, monkeypatch, m, k, n, otherwise):  # noqa: F811
    rng = np.random.default_rng(k + n)
    B = rng.standard_normal((k, n), dtype=np.float32)
    one = np.zeros((m, k), np.float32)
    one[np.arange(m), rng.integers(0, k, m)] = rng.standard_normal(m, dtype=np.float32)
    for A in (rng.standard_normal((m, k), dtype=np.float32), one):
        ref, err = A.astype(np.float64) @ B.astype(np.float64), {}
        for which in (None, otherwise):
            monkeypatch.delenv("CBM_GEMM_SPLIT", raising=False) if which is None else monkeypatch.setenv("CBM_GEMM_SPLIT", which)
            err[which] = np.linalg.norm(_product(env, A, B) - ref)
        assert err[None] <= 1.03 * err[otherwise], err  # (3 %: as many roundings in each as above)
    monkeypatch.delenv("CBM_GEMM_SPLIT", raising=False)
    A = rng.integers(-9, 10, (m, k)).astype(np.float32)
    B = rng.integers(-9, 10, (k, n)).astype(np.float32)
    A[m - 3, k - 1], A[16, 0], B[1, n - 1] = np.inf, np.nan, -np.inf
    with np.errstate(invalid="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.array_equal(_product(env, A, B), ref, equal_nan=True)


@pytest.mark.parametrize("m,k,n", [(132534, 100, 47), (132534, 256, 64), (20000, 500, 64), (50000, 300, 33)])
def test_values_that_are_not_finite_cost_little(env, m, k, n):  # noqa: F811
    """An infinity in B, which reaches one tile of columns in every row: 1.6 to 1.9 times the product's time (measured), the line is at 3.  NaN everywhere: 2.8 to 4.0
    times, the line is at 6.  (Waves that go over all of K alone: 5.2 to 7.3 and 8.4 to 10.7 times where waves share K.)"""
    torch, cbm = env
    A, B, C = torch.randn(m, k, device="cuda"), torch.randn(k, n, device="cuda"), torch.empty(m, n, device="cuda")

    def best():
        us = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                cbm.cbm_dense_matmul(A, B, C)
            b.record()
            torch.cuda.synchronize()
            us.append(a.elapsed_time(b))
        return min(us)

    best()
    clean = best()
    B[3, 2] = float("inf")
    assert best() <= 3 * clean
    A.fill_(float("nan"))
    assert best() <= 6 * clean
