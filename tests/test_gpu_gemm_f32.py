"""The training contraction around the edges of its tiles (128 x 256 of C, 32 of k), in every orientation, with operands
that can and cannot be fetched in aligned groups of four, and with numbers that do not split into bf16 parts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _view(rng, rows, cols, contiguous_rows):
    a = rng.standard_normal((rows, cols) if contiguous_rows else (cols, rows)).astype(np.float32)
    return a if contiguous_rows else a.T


@pytest.mark.parametrize("ta", [True, False])
@pytest.mark.parametrize("tb", [True, False])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (4, 8, 4), (128, 256, 32), (129, 257, 33), (127, 255, 31), (132, 260, 36), (256, 512, 64),
                                   (300, 516, 100), (64, 128, 160), (130, 300, 68)])
def test_contraction_at_the_edges_of_its_tiles(M, N, K, ta, tb):
    """Bound: K roundings of a running fp32 sum, 2^-24 of sum |a||b| each.  It finds wrong elements, a missing second part
    of an operand (2^-8 of it) at every K here, and a missing third part (2^-16) up to K = 36; beyond that
    test_sums_of_one_product does, for every step along k (test_contraction_bounds.py emulates both)."""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(M * 31 + N * 7 + K)
    a, b = _view(rng, M, K, ta), _view(rng, K, N, tb)
    c0 = rng.standard_normal((M, N)).astype(np.float32)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    bound = (K + 2) * 2.0 ** -24 * (np.abs(a).astype(np.float64) @ np.abs(b).astype(np.float64)) + 1e-30
    assert np.all(np.abs(B.op_gemm_f32(a, b) - ref) <= bound)
    assert np.all(np.abs(B.op_gemm_f32(a, b, c0) - (ref + c0)) <= bound + 2.0 ** -23 * (np.abs(ref) + np.abs(c0)))


def test_contraction_of_numbers_beyond_bf16():
    """Infinities, NaN and numbers that round to infinity in bf16 give what fp32 multiply-adds give, in their rows and
    columns; everything else is untouched."""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(5)
    a = rng.standard_normal((300, 64)).astype(np.float32)
    b = rng.standard_normal((64, 600)).astype(np.float32)
    a[3, 5] = np.inf
    a[140, 0] = np.nan
    a[200, 7] = 3.4e38
    b[7, :] = 0.25
    b[9, 300] = -np.inf
    got = B.op_gemm_f32(a, b)
    with np.errstate(invalid="ignore", over="ignore"):
        ref = a.astype(np.float64) @ b.astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)].astype(np.float32))
    ok = np.isfinite(ref)
    fin_a, fin_b = np.where(np.isfinite(a), a, 0).astype(np.float64), np.where(np.isfinite(b), b, 0).astype(np.float64)
    bound = 66 * 2.0 ** -24 * (np.abs(fin_a) @ np.abs(fin_b))
    assert np.all(np.abs(got[ok].astype(np.float64) - ref[ok]) <= bound[ok])


@pytest.mark.parametrize("M,N,K", [(5, 7, 1), (130, 300, 40), (128, 256, 192)])
def test_products_and_sums_that_overflow(M, N, K):
    """Finite operands beyond the largest float: infinities of the right sign and no NaN (every sum here has one sign), and
    columns whose sums stay finite are as exact as ever."""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(K)
    a = rng.uniform(0.5, 2.0, (M, K)).astype(np.float32) * np.float32(1e30)
    b = rng.uniform(0.5, 2.0, (K, N)).astype(np.float32) * np.float32(1e30)
    b[:, ::3] *= np.float32(1e-40)
    a[1::2] *= -1
    got = B.op_gemm_f32(a, b)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    over = np.abs(ref) > 3.5e38
    assert np.array_equal(got[over], np.sign(ref[over]).astype(np.float32) * np.float32(np.inf)) and np.any(over)
    fine = np.abs(ref) < 3.3e38
    assert np.all(np.abs(got[fine] - ref[fine]) <= (K + 2) * 2.0 ** -24 * np.abs(ref[fine]))


@pytest.mark.parametrize("sa,sb", [(1e-36, 1e30), (1e-38, 1e20), (1e-42, 1e20), (1e-44, 1e36), (1e30, 1e-42), (1e-30, 1e-30), (3e31, 1e-8), (1e13, 1e13)])
def test_operands_of_any_size(sa, sb):
    """Operands down to the smallest subnormal numbers and beyond the range that is split into parts: the bound of
    ordinary ones, and the spacing of subnormal results.  (1e36: five deviations of a sum of 200 products stay below 1e38.)"""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(11)
    for M, N, K in ((150, 300, 36), (40, 20, 200)):
        a = (rng.standard_normal((M, K)) * sa).astype(np.float32)
        b = (rng.standard_normal((K, N)) * sb).astype(np.float32)
        a[::7] = rng.standard_normal(a[::7].shape).astype(np.float32)       # rows of ordinary size in the same tiles
        a64, b64 = a.astype(np.float64), b.astype(np.float64)
        with np.errstate(over="ignore"):
            got = B.op_gemm_f32(a, b).astype(np.float64)
        bound = (K + 2) * 2.0 ** -24 * (np.abs(a64) @ np.abs(b64)) + 2.0 ** -149
        assert np.all(np.abs(got - a64 @ b64) <= bound)


@pytest.mark.parametrize("ta", [True, False])
@pytest.mark.parametrize("M,N,K", [(300, 500, 1), (300, 500, 1000), (130, 260, 161), (64, 300, 68)])
def test_sums_of_one_product(M, N, K, ta):
    """One number that is not zero per row of A, so that a result is one product, whatever K: rounded once for K = 1, and
    else within 2^-24 for the rounding and 2^-24 for the products of small parts that are left out.  (An operand's
    third part missing anywhere along k would be an error of up to 2^-17.)"""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(K)
    a = np.zeros((M, K), np.float32)
    a[np.arange(M), rng.integers(0, K, M)] = rng.standard_normal(M)
    b = _view(rng, K, N, True)
    got = B.op_gemm_f32(a if ta else np.ascontiguousarray(a.T).T, b).astype(np.float64)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    assert np.all(np.abs(got - ref) <= (2.0 ** -24 if K == 1 else 2.0 ** -23) * np.abs(ref))


def test_sums_are_as_exact_as_the_fp32_instruction_makes_them():
    """Relative 2-norm of the error over normal numbers: a running fp32 sum, rounded K / 2 times (the fp32 matrix instruction
    adds two products at once), has about 2^-24 / sqrt(3) * sqrt(K / 4) of it (measured 1.15e-6 at K = 4096, 2.0e-7 at
    128); half of that is asked for."""
    from paper_2404_18911_amd import binding as B
    rng = np.random.default_rng(3)
    for K in (128, 1024, 4096):
        a, b = _view(rng, 192, K, True), _view(rng, K, 320, False)
        ref = a.astype(np.float64) @ b.astype(np.float64)
        err = np.linalg.norm(B.op_gemm_f32(a, b) - ref) / np.linalg.norm(ref)
        assert err <= 0.5 * 2.0 ** -24 / 3 ** 0.5 * (K / 4) ** 0.5, (K, err)
