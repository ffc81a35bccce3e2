"""The stand-alone projection over the forms of its input: every row count, K of whole and half k-steps, fewer
k-steps than waves, rows that are 16-byte aligned and rows that are not (another load path, the same sums)."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M,N,K", [(1, 16, 16), (2, 48, 48), (3, 64, 272), (4, 1024, 688), (5, 128, 2064), (8, 256, 4096), (7, 4112, 1040)])
def test_linear_of_aligned_and_unaligned_rows(dtype, M, N, K):
    import torch
    from paper_2404_18911_amd import binding as B
    L = B.lib()
    rng = np.random.default_rng(M * 1000 + K)
    wf = (rng.standard_normal((N, K)) * 0.05).astype(np.float32)
    wh = I.f32_to_bf16_bits(wf) if dtype == "bf16" else wf
    x = rng.standard_normal((M, K)).astype(np.float32)
    code = 1 if dtype == "bf16" else 0
    w = torch.from_numpy(wh.view(np.int16) if code else wh).cuda()
    packed = torch.empty(L.kg_op_packed_bytes(code, N, K), dtype=torch.uint8, device="cuda")
    work = torch.empty(L.kg_op_work_bytes(K), dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    assert L.kg_op_pack(code, w.data_ptr(), N, K, packed.data_ptr(), s) == B.KG_OK
    got = []
    for off in (0, 1):
        buf = torch.full((M * K + 1,), float("nan"), device="cuda")
        xd = buf[off:off + M * K]
        xd.copy_(torch.from_numpy(x.reshape(-1)))
        y = torch.full((M + 1, N), 7.0, device="cuda")
        assert L.kg_op_linear(code, packed.data_ptr(), N, K, xd.data_ptr(), M, y.data_ptr(), work.data_ptr(), s) == B.KG_OK
        torch.cuda.synchronize()
        assert bool((y[M] == 7.0).all())
        got.append(y[:M].cpu().numpy())
    np.testing.assert_array_equal(got[0], got[1])
    w64 = (I.bf16_bits_to_f32(wh) if code else wf).astype(np.float64)
    ref = x.astype(np.float64) @ w64.T
    # rows in two bf16 parts: 2^-17 of a product; float32 sums
    bound = (np.abs(x).astype(np.float64) @ np.abs(w64).T) * 2.0 ** -15 + 1e-7
    assert np.all(np.abs(got[0] - ref) <= bound)


@pytest.mark.parametrize("N,K", [(12288, 528), (13840, 1040), (16400, 528), (19968, 1040), (27648, 272), (22016, 4096), (28688, 272), (32768, 1040),
                                 (12288, 2576), (20480, 2064), (16384, 6160)])
def test_a_row_of_linear_does_not_depend_on_the_others(N, K):
    """6 .. 8 rows (7 and 8 of the second shape, 8 of the seventh and eighth) through 3, 4, 5, 5, 7, 6, 8, 8, 3, 5 and 4 weight tiles per workgroup (256
    compute units), 5 rows too of the last, give the bits of one row alone (uneven shares of tiles, k ranges of unequal length, a half k-step; as many steps as are in flight
    at once, and fewer than twice as many)."""
    import torch
    from paper_2404_18911_amd import binding as B
    L = B.lib()
    g = torch.Generator(device="cuda").manual_seed(N + K)
    w = (torch.randn(N, K, generator=g, device="cuda") * 0.05).bfloat16()
    x = torch.randn(8, K, generator=g, device="cuda")
    packed = torch.empty(L.kg_op_packed_bytes(1, N, K), dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    assert L.kg_op_pack(1, w.data_ptr(), N, K, packed.data_ptr(), s) == B.KG_OK

    def linear(rows):
        y = torch.full((rows.shape[0], N), float("nan"), device="cuda")
        assert L.kg_op_linear(1, packed.data_ptr(), N, K, rows.data_ptr(), rows.shape[0], y.data_ptr(), packed.data_ptr(), s) == B.KG_OK
        return y
    one = torch.cat([linear(x[m:m + 1]) for m in range(8)])
    for M in (5, 6, 7, 8):
        assert torch.equal(linear(x[:M]), one[:M])
    ref = x.double() @ w.double().T
    bound = (x.abs().double() @ w.abs().double().T) * 2.0 ** -15 + 1e-7
    assert bool(((one.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("N,K", [(16, 16), (48, 64), (64, 80), (256, 256), (256, 688), (2048, 1024), (64, 8192)])
def test_a_row_of_an_fp32_product_does_not_depend_on_the_others(N, K):
    """One row goes through the vector units, 2 .. 4 and 5 .. 8 rows through the matrix units: the same bits, also of numbers whose products are
    subnormal or near the top of the range (fewer steps than waves, a last step of 16 k, every number of steps per wave below its ring)."""
    import torch
    from paper_2404_18911_amd import binding as B
    L = B.lib()
    g = torch.Generator(device="cuda").manual_seed(N + K)
    s = torch.cuda.current_stream().cuda_stream
    w = torch.randn(N, K, generator=g, device="cuda") * 0.05
    work = torch.empty(L.kg_op_work_bytes(K), dtype=torch.uint8, device="cuda")

    def linear(rows):
        y = torch.full((rows.shape[0], N), float("nan"), device="cuda")
        assert L.kg_op_linear(0, w.data_ptr(), N, K, rows.data_ptr(), rows.shape[0], y.data_ptr(), work.data_ptr(), s) == B.KG_OK
        return y
    for scale in (1.0, 1e-38, 1e30):
        x = torch.randn(8, K, generator=g, device="cuda") * scale
        one = torch.cat([linear(x[m:m + 1]) for m in range(8)])
        for M in range(2, 9):
            assert torch.equal(linear(x[:M]), one[:M]), (scale, M)
        ref = x.double() @ w.double().T
        bound = (x.abs().double() @ w.abs().double().T) * (K + 8) * 2.0 ** -24 + K * 1.5e-45       # K + 8 roundings of a sum, and of subnormal products
        assert bool(((one.double() - ref).abs() <= bound).all()), scale


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_of_more_than_two_gib(dtype):
    """Eight rows whose last lies beyond 2^31 bytes: the bits of that row alone."""
    import torch
    from paper_2404_18911_amd import binding as B
    L, code = B.lib(), 1 if dtype == "bf16" else 0
    N, K = 16, 76_800_000
    s = torch.cuda.current_stream().cuda_stream
    w = torch.empty(N, K, dtype=torch.bfloat16 if code else torch.float32, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(1))
    packed = torch.empty(L.kg_op_packed_bytes(code, N, K), dtype=torch.uint8, device="cuda")
    assert L.kg_op_pack(code, w.data_ptr(), N, K, packed.data_ptr(), s) == B.KG_OK
    x = torch.empty(8, K, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(2))
    y, one = torch.full((8, N), 7.0, device="cuda"), torch.full((8, N), 7.0, device="cuda")
    assert L.kg_op_linear(code, packed.data_ptr(), N, K, x.data_ptr(), 8, y.data_ptr(), packed.data_ptr(), s) == B.KG_OK
    for m in (0, 6, 7):
        assert L.kg_op_linear(code, packed.data_ptr(), N, K, x[m].data_ptr(), 1, one[m].data_ptr(), packed.data_ptr(), s) == B.KG_OK
        assert torch.equal(y[m], one[m]), m
    ref = (x[7].double() * w[3].double()).sum()
    assert abs(float(y[7, 3] - ref)) <= 1e-3 * K ** 0.5         # (sums of 7.7e7 products: their spread is K^0.5)
