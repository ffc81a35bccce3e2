"""The stand-alone projection where its output shares memory with its input, wholly or in part: the bits of a call with
memory of its own, for both entry points, eagerly and on every replay of a captured graph.  Enough workgroups that some
would write y while others still read x (256 compute units, several rounds of workgroups)."""
import pytest

pytestmark = pytest.mark.gpu


def _setup(dtype, N, K, seed):
    import torch
    from paper_2404_18911_amd import binding as B
    L = B.lib()
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.randn(N, K, generator=g, device="cuda") * K ** -0.5
    w = w.bfloat16() if dtype else w
    packed = torch.empty(L.kg_op_packed_bytes(dtype, N, K), dtype=torch.uint8, device="cuda")
    work = torch.empty(L.kg_op_work_bytes(K), dtype=torch.uint8, device="cuda")
    assert L.kg_op_pack(dtype, w.data_ptr(), N, K, packed.data_ptr(), torch.cuda.current_stream().cuda_stream) == B.KG_OK

    def call(static, x_ptr, M, y_ptr, stream=None):
        s = stream if stream is not None else torch.cuda.current_stream().cuda_stream
        rc = L.kg_op_linear_static(dtype, packed.data_ptr(), N, K, x_ptr, M, y_ptr, s) if static else \
            L.kg_op_linear(dtype, packed.data_ptr(), N, K, x_ptr, M, y_ptr, work.data_ptr(), s)
        assert rc == B.KG_OK
    return torch, g, call, (packed, work)


# y's first element minus x's, in floats: the same memory; y behind x's first row, also unaligned; y ending inside x;
# y touching x's last float only; y right behind x and right before it (no overlap)
@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("dtype,N,K,M", [(1, 8192, 8192, 1), (1, 8192, 8192, 8), (1, 12288, 1040, 7), (0, 4096, 4096, 3), (1, 272, 16384, 8)])
def test_output_in_the_memory_of_the_input(static, dtype, N, K, M):
    torch, g, call, keep = _setup(dtype, N, K, N + K + M)
    x = torch.randn(M, K, generator=g, device="cuda")
    want = torch.empty(M, N, device="cuda")
    call(False, x.data_ptr(), M, want.data_ptr())
    for off in (0, K, 1, -1, -(M * N) + 1, M * K - 1, M * K, -(M * N)):
        x0 = max(0, -off)
        buf = torch.full((x0 + max(M * K, off + M * N),), float("nan"), device="cuda")
        buf[x0:x0 + M * K] = x.reshape(-1)
        call(static, buf.data_ptr() + 4 * x0, M, buf.data_ptr() + 4 * (x0 + off))
        got = buf[x0 + off:x0 + off + M * N].reshape(M, N)
        assert torch.equal(got, want), off
    del keep


def test_in_place_call_in_a_captured_graph():
    """x <- W x, replayed: every replay against the eager product of what the replay before it left."""
    N = K = 4096
    torch, g, call, keep = _setup(1, N, K, 9)
    x = torch.randn(1, K, generator=g, device="cuda")
    state = x.clone()
    call(True, state.data_ptr(), 1, state.data_ptr())                     # (the array's address is looked up outside the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(True, state.data_ptr(), 1, state.data_ptr(), torch.cuda.current_stream().cuda_stream)
    state.copy_(x)
    for _ in range(4):
        before, want = state.clone(), torch.empty(1, N, device="cuda")
        call(False, before.data_ptr(), 1, want.data_ptr())
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(state, want)
    del keep
