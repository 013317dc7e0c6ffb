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
            # K additions of 2^-24 each, and parts left out below 2^-24 of a term (three pairs at most)
            bound = (2 * k + 8) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64))
            assert np.all(np.abs(got - ref) <= bound + 1e-37), (n, pad)
            Ai, Bi = (rng.integers(-9, 10, s).astype(np.float32) for s in ((m, k), (k, n)))
            assert np.array_equal(_product(env, Ai, Bi, pad).astype(np.float64), Ai.astype(np.float64) @ Bi.astype(np.float64))


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


@pytest.mark.parametrize("n", [16, 17, 47, 112, 130])
def test_panel_kernel_on_any_b(env, monkeypatch, n):
    monkeypatch.setenv("CBM_GEMM_SPLIT", "0")
    rng = np.random.default_rng(n)
    m, k = 8193, 36   # just tall enough for the panel kernel
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
