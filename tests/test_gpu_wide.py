"""Models 8064 and 8192 features wide, whose long projections keep one chunk of weights in flight per wave: verification rows against one-token
decoding bit for bit, and both against the prompt pass, which goes through other kernels."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [63, 64])
def test_rows_of_wide_projections(heads):
    """(2e-3 of the logits' spread between the passes: the bound of the other prompt tests)"""
    import torch
    from paper_2404_18911_amd import binding as B
    shape = I.ModelShape("wide", 1, 128 * heads, heads, 128, 5120, 9216, 1)
    kg = B.Kangaroo(shape, 64, gamma_max=7, kv_page_tokens=16)
    g = torch.Generator(device="cuda").manual_seed(heads)
    for kind, layer, r, c in I.tensor_list(shape):
        norm = r == 1
        t = (torch.ones(c, device="cuda") if norm else torch.randn(r, c, generator=g, device="cuda") * (1.0 if kind == I.KIND_EMBED else 0.01)).bfloat16()
        kg._chk(kg.L.kg_load_tensor(kg.h, kind, layer, t.data_ptr(), t.numel()))
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, 20, seed=6)]
    for gamma in (1, 2, 3, 4, 5, 6):
        p, _ = B.make_params(eta=0.0, gamma=gamma)
        chain = [kg.prefill(p, prompt)]
        for _ in range(gamma):
            chain.append(kg.draft_step(p)[0])
        tokens = kg.verify(p)
        rows = [kg.read_logits(1, r) for r in range(gamma + 1)]
        kg.prefill(p, prompt)
        for r, t in enumerate(chain):
            assert kg.plain_step(p, t) == tokens[r]
            np.testing.assert_array_equal(rows[r], kg.read_logits(1, 0))
        kg.prefill(p, prompt + chain)
        np.testing.assert_allclose(kg.read_logits(1, 0), rows[-1], rtol=0, atol=2e-3 * max(1.0, float(np.std(rows[-1]))))
    kg.close()
