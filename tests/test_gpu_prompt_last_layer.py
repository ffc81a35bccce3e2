"""The last layer of a prompt pass computes keys and values for every row and the rest for the last row only: logits and every cache against
the same tokens fed one at a time, where that row's query comes from (a pass of up to 384 rows takes it from the projection of all
rows, a longer one computes it by itself) and how many passes the prompt has, with every cache type and with the exit at the last layer."""
import dataclasses

import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu

BASE = I.ModelShape("last_layer", 3, 512, 8, 64, 1384, 1024, 1)
# 1024 rows a pass with the bf16 and f32 caches, 4096 with the half-precision one
LENGTHS = {"f16": [9, 15, 16, 193, 384, 385, 1023, 4096, 4097, 4480, 4481], "bf16": [2, 9, 385, 1024, 1025, 1033], "f32": [2, 9, 385, 1024, 1025]}


@pytest.mark.parametrize("exit_layer", [1, 3])
@pytest.mark.parametrize("kv", ["f16", "bf16", "f32"])
def test_prompts_agree_with_one_token_decoding(kv, exit_layer):
    """Bounds with the half-precision cache as in test_prompt_pass_agrees_with_one_token_decoding (a value may round to the neighbouring
    half, 2^-11 relative, what lies upstream of it moves by as much; logits 2e-3); bit for bit with the others."""
    import torch
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = dataclasses.replace(BASE, kv=kv, exit_layer=exit_layer)
    W = I.gen_weights(shape, seed=11, alpha=1.0)
    lengths = LENGTHS[kv]
    n = max(lengths)
    prompt = [int(t) for t in I.gen_prompt(shape.vocab, n, seed=12)]
    kg = P.load_model(shape, W, n + 16)
    p, _ = B.make_params()
    kg.prefill(p, prompt[:1])
    logits = {}
    for i in range(1, n):
        kg.plain_step(p, prompt[i])
        if i + 1 in lengths:
            logits[i + 1] = kg.read_logits(1, 0)
    at = [0, 7, 8, 127, 128, 383, 384, 1023, 1024, 4095, 4096]
    slots = range(shape.n_layers)
    want = {(s, i): np.stack(kg.read_kv(s, i)) for s in slots for i in at + [m - 1 for m in lengths] if i < n}
    for m in lengths:
        kg.kv.fill_(0xFF)           # not a number in every cache type
        kg.prefill(p, prompt[:m])
        z = kg.read_logits(1, 0)
        got = {(s, i): np.stack(kg.read_kv(s, i)) for s, i in want if i < m}
        if kv == "f16":
            np.testing.assert_allclose(z, logits[m], rtol=0, atol=2e-3 * max(1.0, float(np.std(logits[m]))), err_msg=str(m))
        else:
            np.testing.assert_array_equal(z, logits[m], err_msg=str(m))
        for key, g in got.items():
            if kv == "f16":
                assert float((np.abs(g - want[key]) / (np.abs(want[key]) + 1.0)).max()) <= 2e-3, (m, key)
            else:
                np.testing.assert_array_equal(g, want[key], err_msg=str((m, key)))
    kg.close()
