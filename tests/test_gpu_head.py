"""The LM head over verification rows where several weight tiles share a workgroup (6 rows and more, vocabularies of 3 to 8
tiles per compute unit): the logits and choices of one-token decoding, bit for bit."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [8208, 12288, 16384, 16400, 24576, 28672, 32000])
def test_verification_rows_through_the_head_equal_decoded_rows(vocab):
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("head", 2, 512, 8, 64, 1376, vocab, 1)
    W = I.gen_weights(shape, seed=4, alpha=1.0)
    kg = P.load_model(shape, W, 64, gamma_max=7, kv_page_tokens=16)
    prompt = [int(t) for t in I.gen_prompt(vocab, 12, seed=2)]
    for gamma in (3, 4, 5, 6, 7):
        p, _ = B.make_params(eta=0.0, gamma=gamma)
        chain = [kg.prefill(p, prompt)]
        for _ in range(gamma):
            chain.append(kg.draft_step(p)[0])
        tokens = kg.verify(p)
        rows = [kg.read_logits(1, r) for r in range(gamma + 1)]
        assert len(tokens) == gamma + 1
        assert kg.prefill(p, prompt) == chain[0]
        for r, t in enumerate(chain):
            assert kg.plain_step(p, t) == tokens[r]
            one = kg.read_logits(1, 0)
            np.testing.assert_array_equal(rows[r], one)
            assert tokens[r] == int(np.argmax(one))
    kg.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab", [16, 1024, 16384, 16400, 131072, 131088, 147472])
def test_choices_draws_and_confidences_follow_the_logits(vocab, dtype):
    """From one weight tile to more than eight per thread of the final reduction (which keeps eight in registers): the arg-max, the token that
    a uniform number draws and the confidence against the row's logits in 64 bits.  A draw may fall to a neighbour where the number lies within
    1e-5 of a boundary (float32 tile sums of 16 exponentials: 2^-20)."""
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("vocab", 2, 64, 1, 64, 64, vocab, 1, dtype)
    W = I.gen_weights(shape, seed=9, alpha=1.0, head_scale=8.0)
    kg = P.load_model(shape, W, 48, kv_page_tokens=16)
    prompt = [int(t) for t in I.gen_prompt(vocab, 10, seed=3)]

    def parts(z):
        w = np.exp(z.astype(np.float64) - z.max())
        return np.cumsum(w), w.sum()

    def drawn(z, u, tok):
        c, total = parts(z)
        assert (c[tok - 1] if tok else 0.0) - 1e-5 * total <= u * total <= c[tok] + 1e-5 * total, (u, tok)
    greedy, _ = B.make_params(eta=0.0)
    tok = kg.prefill(greedy, prompt)
    assert tok == int(np.argmax(kg.read_logits(1, 0)))
    for i in range(3):
        t, conf, _ = kg.draft_step(greedy)
        z = kg.read_logits(0, i)
        assert t == int(np.argmax(z))
        assert abs(conf * parts(z)[1] - 1.0) <= 1e-5
    for u in (0.0, 0.03, 0.5, 0.97, float(np.float32(1.0 - 2.0 ** -24))):
        table = np.full((48, 3), u, dtype=np.float32)
        p, keep = B.make_params(mode=1, temperature=1.0, eta=0.0, uniforms=table)
        tok = kg.prefill(p, prompt)
        drawn(kg.read_logits(1, 0), u, tok)
        t, _, _ = kg.draft_step(p)
        drawn(kg.read_logits(0, 0), u, t)
    kg.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lowest", [False, True])
def test_logits_of_minus_infinity(dtype, lowest):
    """Rows whose logits all overflow to minus infinity choose the lowest token, as an arg-max with ties does (their sum of weights is 0);
    with one finite logit among them that one, with all the probability."""
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("minus", 1, 64, 1, 64, 64, 1040, 1, dtype)
    W = I.gen_weights(shape, seed=9, alpha=1.0)
    store = (lambda a: a) if dtype == "f32" else I.f32_to_bf16_bits
    # the residual stream is the embedding (8 in its first feature once normalised), and the head reads that feature only
    embed, head = np.zeros((1040, 64), dtype=np.float32), np.zeros((1040, 64), dtype=np.float32)
    embed[:, 0] = 1.0
    head[:, 0] = -3e38
    if lowest:
        head[700, 0] = -3.0
    W[(I.KIND_EMBED, -1)], W[(I.KIND_LM_HEAD, -1)] = store(embed), store(head)
    for k in (I.KIND_WO, I.KIND_WD):
        W[(k, 0)] = np.zeros_like(W[(k, 0)])
    W[(I.KIND_A_WO, -1)] = np.zeros_like(W[(I.KIND_A_WO, -1)])
    kg = P.load_model(shape, W, 48, kv_page_tokens=16)
    want = 700 if lowest else 0
    for mode in (0, 1):
        p, keep = B.make_params(mode=mode, temperature=1.0, eta=0.0, uniforms=np.full((48, 3), 0.5, dtype=np.float32))
        assert kg.prefill(p, [3, 4, 5]) == want
        z = kg.read_logits(1, 0)
        assert np.isneginf(np.delete(z, 700)).all() and np.isneginf(z[700]) != lowest
        t, conf, _ = kg.draft_step(p)
        assert t == want and conf == (1.0 if lowest else np.inf)
        kg.prefill(p, [3, 4, 5])
        assert kg.plain_step(p, want) == want
    kg.close()
