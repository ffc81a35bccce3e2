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
