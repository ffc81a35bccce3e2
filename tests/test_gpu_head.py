"""The LM head over verification rows where several weight tiles share a workgroup (6 rows and more, vocabularies of 3 to 7
tiles per compute unit): the logits and choices of one-token decoding, bit for bit."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [8208, 12288, 16384, 16400, 24576, 28672])
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
