"""Prompt attention in workgroups of 32 and of 128 rows (two widths of heads) with pages shorter than, as long as and longer than a tile of 64
positions, in shuffled order, and with a second pass behind 4096 cached positions: logits against the same tokens fed one at a time."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu

# one layer, whose attention output is what the logits come from; 40 heads reach the large workgroups at 385 rows, 4 heads never
SHAPES = {"narrow": I.ModelShape("narrow_1", 1, 2560, 40, 64, 640, 1024, 1), "wide": I.ModelShape("wide_1", 1, 5120, 40, 128, 640, 1024, 1),
          "few": I.ModelShape("few_1", 1, 512, 4, 128, 640, 1024, 1)}


def _compare(shape, page, lengths):
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    W = I.gen_weights(shape, seed=21, alpha=1.0)
    n = max(lengths)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, n, seed=22)]
    kg = P.load_model(shape, W, n + 16, kv_page_tokens=page)
    order = np.random.default_rng(5).permutation(len(kg.page_order)).astype(np.int32)
    kg.set_page_order(order)
    p, _ = B.make_params()
    kg.prefill(p, prompt[:1])
    want = {1: kg.read_logits(1, 0)}
    for i in range(1, n):
        kg.plain_step(p, prompt[i])
        if i + 1 in lengths:
            want[i + 1] = kg.read_logits(1, 0)
    for m in lengths:
        kg.kv.fill_(0xFF)           # not a number
        kg.prefill(p, prompt[:m])
        z = kg.read_logits(1, 0)
        np.testing.assert_allclose(z, want[m], rtol=0, atol=2e-3 * max(1.0, float(np.std(want[m]))), err_msg=str((page, m)))
    kg.close()


@pytest.mark.parametrize("page", [16, 32, 64, 128])
@pytest.mark.parametrize("name", list(SHAPES))
def test_every_page_size(name, page):
    """(2e-3 of the logits' spread: the bound of the other prompt tests, for values that round to the neighbouring half)"""
    _compare(SHAPES[name], page, [9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 257, 384, 385, 449, 513, 575, 640, 641, 700, 1025])


def test_a_second_pass_behind_4096_positions():
    _compare(SHAPES["few"], 128, [4097, 4111, 4160, 4161])
    _compare(SHAPES["narrow"], 64, [4096, 4096 + 385, 4096 + 449])


def _scaled(bits, by):
    return I.f32_to_bf16_bits(I.bf16_bits_to_f32(bits) * by)


@pytest.mark.parametrize("hd", [64, 128])
def test_a_row_does_not_depend_on_later_ones(hd):
    """Two prompts that differ in the last token leave the same bits in both layers' caches at every earlier position (what a row sees
    decides where the reference of its probabilities lies, not what its neighbours see).  Queries 64 times as large as usual: scores spread so far
    that a late row's maximum often leaves the others' behind."""
    import torch
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("apart", 2, 40 * hd, 40, hd, 640, 1024, 2)
    W = I.gen_weights(shape, seed=31, alpha=1.0)
    for i in range(2):
        W[(I.KIND_WQ, i)] = _scaled(W[(I.KIND_WQ, i)], 64.0)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, 700, seed=32)]
    page = 128
    kg = P.load_model(shape, W, 720, kv_page_tokens=page)
    p, _ = B.make_params()

    def caches(tokens):
        kg.kv.zero_()
        kg.prefill(p, tokens)
        n = 6 * 3 * 40 * 2 * page * hd
        pool = kg.kv.view(torch.int16)[:n].view(6, 3, 40, 2, page, hd)[:, :2].permute(0, 4, 1, 2, 3, 5).reshape(6 * page, -1)
        return pool[:len(tokens) - 1].clone()
    for n in (33, 63, 160, 300, 640, 700):
        want = caches(prompt[:n])
        for last in (1, 500, 1000):
            assert torch.equal(caches(prompt[:n - 1] + [last]), want), (n, last)
    kg.close()


@pytest.mark.parametrize("name", ["narrow", "wide"])
def test_queries_up_to_the_half_precision_range(name):
    """Scaled queries of 55 thousand, which a half holds (and 1.44 times as much it does not): every embedding is a row of signs, so that the
    normalised input is too, and a head's queries are one of its features times a number, at the first rotation pair's first component."""
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = SHAPES[name]
    d, hd = shape.d_model, shape.head_dim
    W = I.gen_weights(shape, seed=41, alpha=1.0)
    W[(I.KIND_EMBED, -1)] = I.f32_to_bf16_bits(np.where(np.random.default_rng(42).random((shape.vocab, d)) < 0.5, -1.0, 1.0).astype(np.float32))
    wq = np.zeros((d, d), dtype=np.float32)
    for h in range(shape.n_heads):
        wq[h * hd, 7 * h] = 55000.0 * np.sqrt(hd)
    W[(I.KIND_WQ, 0)] = I.f32_to_bf16_bits(wq)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, 600, seed=43)]
    kg = P.load_model(shape, W, 616)
    p, _ = B.make_params()
    lengths, want = (9, 40, 200, 600), {}
    kg.prefill(p, prompt[:1])
    for i in range(1, max(lengths)):
        kg.plain_step(p, prompt[i])
        if i + 1 in lengths:
            want[i + 1] = kg.read_logits(1, 0)
    for n in lengths:
        kg.prefill(p, prompt[:n])
        z = kg.read_logits(1, 0)
        assert np.isfinite(z).all(), n
        np.testing.assert_allclose(z, want[n], rtol=0, atol=2e-3 * max(1.0, float(np.std(want[n]))), err_msg=str(n))
    kg.close()


@pytest.mark.parametrize("hd", [64, 128])
def test_the_largest_probability_is_exact(hd):
    """Rows that see one position at about 149 times the weight of another one, read by the same wave many positions earlier, and nothing else: where both
    values are 1 the output is 1 but for the half-precision rounding of the smaller probability (0.0067 x 2^-12) and the two bfloat16 parts
    of the output (2^-17), together below 2^-16.  (The larger one, rounded relative to the smaller: 2.5e-4.)  Workgroups of 32 and of 128 rows."""
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    d = 40 * hd
    # (a base of the rotation so large that the pair used here does not turn)
    shape = I.ModelShape("exact", 2, d, 40, hd, 640, 1024, 1, rope_theta=1e12)
    W = I.gen_weights(shape, seed=51, alpha=1.0)
    rng = np.random.default_rng(52)
    # features of a token: 1, the signs that mark tokens 0 and 1, random signs: the normalised input is the same
    embed = np.where(rng.random((shape.vocab, d)) < 0.5, -1.0, 1.0).astype(np.float32)
    embed[:, 0], embed[:, 1:3] = 1.0, -1.0
    embed[0, 1] = embed[1, 2] = 1.0
    wq, wk = np.zeros((d, d), dtype=np.float32), np.zeros((d, d), dtype=np.float32)
    at = np.arange(40) * hd + hd // 2 - 1
    wq[at, 0] = np.sqrt(hd)
    wk[at, 1], wk[at, 2] = 24.0, 26.5           # keys -2.5, 2.5 and -50.5 of tokens 0, 1 and others
    for kind, a in ((I.KIND_EMBED, embed), (I.KIND_WQ, wq), (I.KIND_WK, wk), (I.KIND_WV, np.eye(d, dtype=np.float32)),
                    (I.KIND_WO, np.eye(d, dtype=np.float32)), (I.KIND_WD, np.zeros((d, 640), dtype=np.float32))):
        W[(kind, -1 if kind == I.KIND_EMBED else 0)] = I.f32_to_bf16_bits(a)
    kg = P.load_model(shape, W, 720)
    kg.train_bind(704)
    for n in (200, 700):
        tokens = [0] + [int(t) for t in rng.integers(2, 1024, n - 1)]
        tokens[140] = 1                         # (in the fifth tile of 32: the same wave's as the first)
        F, _ = kg.train_features(tokens)
        out = (F.cpu().numpy() - embed[tokens])[140:, (embed[0] == 1.0) & (embed[1] == 1.0)]
        assert out.shape[1] > 200 and np.abs(out - 1.0).max() <= 2.0 ** -16, np.abs(out - 1.0).max()
    kg.close()
