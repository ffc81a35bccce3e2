"""Prompt passes of every length class against the same tokens fed one at a time through the decode
kernels: the half-precision cache and the logits after each prompt length.  Shapes: the 7B and 13B layer
widths (they reach every number of weight tiles per workgroup) and a narrow one whose feed-forward width
is no multiple of 32 and whose k-steps do not divide by the eight k ranges of a weight tile row, and one whose
down_proj has more than 1024 k-steps."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu

SHAPES = {
    "7b": I.ModelShape("7b_1", 1, 4096, 32, 128, 11008, 1024, 1),
    "13b": I.ModelShape("13b_1", 1, 5120, 40, 128, 13824, 1024, 1),
    "uneven": I.ModelShape("uneven_2", 2, 1344, 21, 64, 3416, 1024, 1),
    "long": I.ModelShape("long_1", 1, 512, 8, 64, 33800, 1024, 1),
}
# around the edges of 16-row pairs, of the row groups of the stream kernel (16, 32, 48, 64, 96, 128 rows), of its range
# (9 .. 96 rows at d_model 4096, .. 192 in narrow models) and of the decode kernels' (8 rows); then longer passes, which take every tile
# size, row group (80, 96, 112, 128 rows) and number of slices along k of the larger kernels, with last row groups of one row, of a
# pair and a row, and of a whole group but one row
LENGTHS = [1, 8, 9, 16, 17, 31, 33, 48, 49, 64, 65, 96, 97, 112, 113, 128, 129, 160, 161, 192, 193, 241, 256, 257, 289, 300, 337, 385, 401, 511, 561,
           777, 1025, 1465, 2001, 3001]


@pytest.fixture(scope="module", params=list(SHAPES))
def reference(request):
    """A model, its prompt, and cache and logits after each token from one-token decoding."""
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    import torch
    shape = SHAPES[request.param]
    W = I.gen_weights(shape, seed=5, alpha=1.0)
    n = max(LENGTHS)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, n, seed=6)]
    kg = P.load_model(shape, W, n + 16)
    p, _ = B.make_params()
    kg.prefill(p, prompt[:1])
    logits = {1: kg.read_logits(1, 0)}
    for i in range(1, n):
        kg.plain_step(p, prompt[i])
        if i + 1 in LENGTHS:
            logits[i + 1] = kg.read_logits(1, 0)
    torch.cuda.synchronize()
    cache = _cache(kg, shape).clone()
    yield shape, kg, p, prompt, cache, logits
    kg.close()


def _cache(kg, shape):
    """[cache][head][K|V][position][dimension] of the model's layers, float32."""
    import torch
    P, H, hd, slots = kg.cfg.kv_page_tokens, shape.n_heads, shape.head_dim, shape.n_layers + 1
    pages = len(kg.page_order)
    pool = kg.kv.view(torch.float16)[: pages * slots * H * 2 * P * hd].view(pages, slots, H, 2, P, hd)[:, : shape.n_layers]
    return pool.permute(1, 2, 3, 0, 4, 5).reshape(shape.n_layers, H, 2, pages * P, hd).float()


@pytest.mark.parametrize("n", LENGTHS)
def test_a_prompt_of_n_tokens_agrees_with_one_token_decoding(reference, n):
    """Bounds as in test_prompt_pass_agrees_with_one_token_decoding: a value may round to the neighbouring half
    (2^-11 relative), what lies upstream of it moves by as much; logits 2e-3."""
    import torch
    shape, kg, p, prompt, cache, logits = reference
    kg.kv.view(dtype=torch.float16).fill_(float("nan"))
    kg.prefill(p, prompt[:n])
    got, want = _cache(kg, shape)[:, :, :, :n], cache[:, :, :, :n]
    err = float(((got - want).abs() / (want.abs() + 1.0)).max())
    assert err <= 2e-3, err
    z = kg.read_logits(1, 0)
    np.testing.assert_allclose(z, logits[n], rtol=0, atol=2e-3 * max(1.0, float(np.std(logits[n]))))


@pytest.mark.parametrize("max_seq", [24, 40, 200, 296, 344, 776])
def test_a_prompt_that_fills_the_context_s_last_block(max_seq):
    """Contexts of an odd number of 8-row blocks, filled to the last row a prompt may have: the last block has no partner in
    the pair layout of the activations.  Every cache, the adapter's included, and the logits agree with the same prompt in
    a context with room to spare, bit for bit, and no byte behind the scratch buffer changes."""
    import torch
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = SHAPES["uneven"]
    W = I.gen_weights(shape, seed=5, alpha=1.0)
    p, _ = B.make_params(gamma=1)
    n = max_seq - 3
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, n, seed=7)]
    got = []
    for room in (0, 136):
        kg = P.load_model(shape, W, max_seq + room, gamma_max=1)
        guard = torch.full((kg.scratch_bytes + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
        kg.scratch = guard[:kg.scratch_bytes]
        kg._chk(kg.L.kg_bind(kg.h, kg.arena.data_ptr(), kg.weight_bytes, kg.kv.data_ptr(), kg.kv_bytes, kg.scratch.data_ptr(),
                             kg.scratch_bytes, kg.stream.cuda_stream))
        kg.load_weights((k, l, W[(k, l)]) for k, l, _, _ in I.tensor_list(shape))
        kg.kv.zero_()
        token = kg.prefill(p, prompt)
        torch.cuda.synchronize()
        assert bool((guard[kg.scratch_bytes:] == 0xA5).all())
        got.append((token, kg.read_logits(1, 0), [kg.read_kv(s, i) for s in range(shape.n_layers + 1) for i in (0, 1, 7, 8, 15, 16, n // 2, n - 1)]))
        kg.close()
    assert got[0][0] == got[1][0]
    np.testing.assert_array_equal(got[0][1], got[1][1])
    for a, b in zip(got[0][2], got[1][2]):
        np.testing.assert_array_equal(np.stack(a), np.stack(b))
