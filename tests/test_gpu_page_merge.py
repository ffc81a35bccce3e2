"""Rows of a verification pass whose launch covers nine pages or more while the earlier ones attend to eight: logits, cached keys and values
of one-token decoding, bit for bit, since neither the other rows nor the trailing pages of a launch may show in a row."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


def _check(hd, kv, page, start, rows):
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("pages", 2, 512, 512 // hd, hd, 1376, 1024, 1, kv=kv)
    W = I.gen_weights(shape, seed=14, alpha=1.0)
    top = max(start) + max(rows)
    kg = P.load_model(shape, W, top + 16, gamma_max=7, kv_page_tokens=page)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, max(start), seed=15)]

    def cached(at, n):
        return [np.stack(kg.read_kv(s, i)) for s in range(shape.n_layers) for i in range(at, at + n)]
    for at in start:
        for n in rows:
            p, _ = B.make_params(eta=0.0, gamma=n - 1)
            chain = [kg.prefill(p, prompt[:at])]
            for _ in range(n - 1):
                chain.append(kg.draft_step(p)[0])
            tokens = kg.verify(p)
            logits, kvs = [kg.read_logits(1, r) for r in range(n)], cached(at, n)
            assert kg.prefill(p, prompt[:at]) == chain[0]
            for r, t in enumerate(chain):
                assert kg.plain_step(p, t) == tokens[r]
                np.testing.assert_array_equal(logits[r], kg.read_logits(1, 0), err_msg=str((at, n, r)))
            for a, b in zip(kvs, cached(at, n)):
                np.testing.assert_array_equal(a, b, err_msg=str((at, n)))
    kg.close()


@pytest.mark.parametrize("kv", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("hd", [64, 128])
def test_rows_before_and_behind_the_ninth_page(hd, kv):
    """Position 128 with pages of 16; 512 too, where 33 pages are more than are asked for at once."""
    _check(hd, kv, 16, [121, 124, 127], range(2, 9))
    _check(hd, kv, 16, [509], [2, 4, 5, 8])


def test_rows_before_and_behind_position_1024_with_pages_of_128():
    _check(128, "f16", 128, [1021, 1023], [2, 4, 8])
