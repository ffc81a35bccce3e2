"""What the bounds of test_gpu_gemm_f32.py tell apart: the contraction's arithmetic (three bf16 parts of an operand, six of
their nine products, those of the first parts in a sum of their own) emulated in numpy, as it is and with mistakes planted
into the emulation."""
import numpy as np
import pytest

SCALE = np.float32(2.0 ** 24)
PRODUCTS = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def _bf16(x):
    b = x.view(np.uint32).astype(np.uint64)
    return (((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(np.float32)


def _parts(x):
    out, r = [], np.ascontiguousarray(x) * SCALE
    for _ in range(3):
        out.append(_bf16(r))
        r = r - out[-1]
    return out


def _contract(a, b, products=PRODUCTS, steps=None):
    """steps: the 32-wide steps along k in which only `products` are taken (all six elsewhere); None: everywhere."""
    pa, pb = _parts(a), _parts(b)
    k = np.arange(a.shape[1])
    main, rest = (np.zeros((a.shape[0], b.shape[1]), np.float32) for _ in range(2))
    for i, j in sorted(PRODUCTS, key=lambda p: -sum(p)):
        on = np.ones(len(k), bool) if (i, j) in products else (np.zeros(len(k), bool) if steps is None else ~np.isin(k // 32, steps))
        for k0 in range(0, len(k), 16):
            s = slice(k0, k0 + 16)
            t = (pa[i][:, s] * on[s]).astype(np.float64) @ pb[j][s].astype(np.float64)
            if i + j:
                rest = (rest + t).astype(np.float32)
            else:
                main = (main + t).astype(np.float32)
    return (main + rest) * np.float32(2.0 ** -48)


def _edge_bound_holds(got, a, b):
    a64, b64, K = a.astype(np.float64), b.astype(np.float64), a.shape[1]
    return bool(np.all(np.abs(got - a64 @ b64) <= (K + 2) * 2.0 ** -24 * (np.abs(a64) @ np.abs(b64)) + 1e-30))


def _one_product_bound_holds(got, a, b):
    ref = a.astype(np.float64) @ b.astype(np.float64)
    return bool(np.all(np.abs(got - ref) <= 2.0 ** -23 * np.abs(ref)))


@pytest.mark.parametrize("M,N,K", [(128, 256, 32), (132, 260, 36), (300, 516, 100), (64, 128, 160)])
def test_the_edge_test_accepts_the_arithmetic_and_finds_a_missing_second_part(M, N, K):
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    a, b = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    assert _edge_bound_holds(_contract(a, b), a, b)
    assert not _edge_bound_holds(_contract(a, b, [p for p in PRODUCTS if p[0] != 1]), a, b)
    assert not _edge_bound_holds(_contract(a, b, [p for p in PRODUCTS if p[1] != 1]), a, b)
    if K <= 36:
        assert not _edge_bound_holds(_contract(a, b, [p for p in PRODUCTS if 2 not in p]), a, b)


@pytest.mark.parametrize("M,N,K", [(300, 500, 1000), (130, 260, 161), (64, 300, 68)])
def test_sums_of_one_product_find_a_missing_product_in_a_single_step(M, N, K):
    rng = np.random.default_rng(K)
    a = np.zeros((M, K), np.float32)
    at = rng.integers(0, K, M)
    a[np.arange(M), at] = rng.standard_normal(M)
    b = rng.standard_normal((K, N)).astype(np.float32)
    assert _one_product_bound_holds(_contract(a, b), a, b)
    for missing in PRODUCTS:
        for step in np.unique(at // 32)[:: max(1, K // 125)]:
            assert not _one_product_bound_holds(_contract(a, b, [p for p in PRODUCTS if p != missing], steps=[step]), a, b), (missing, step)


@pytest.mark.parametrize("x", [1e-45, 3e-42, 1.1754942e-38, 1e-36, 1.0, 2e31])
def test_the_scaled_split_is_exact(x):
    rng = np.random.default_rng(1)
    v = (rng.uniform(0.5, 1.0, 2000) * x).astype(np.float32)
    parts = _parts(v)
    assert np.array_equal(sum(p.astype(np.float64) for p in parts), v.astype(np.float64) * 2.0 ** 24)
    for p in parts:
        assert np.all((p == 0) | (np.abs(p) >= 2.0 ** -126))
