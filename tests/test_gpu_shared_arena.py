"""Several contexts of one model bound to one weight arena: the tiled form of the weights depends on the model alone, not on the
type of a context's cache, so contexts with different caches may share it (every one loads the tensors once; the bytes are the same)."""
import dataclasses

import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu
NEW = 20


def _outputs(kg, prompts):
    from paper_2404_18911_amd import binding as B
    p, _ = B.make_params(eta=0.5, gamma=6)
    out = []
    for prompt in prompts:
        out += [kg.prefill(p, prompt), kg.read_logits(1, 0), *kg.read_kv(1, 3)]
        out += [kg.generate(p, prompt, NEW)[0], kg.read_logits(1, 0), *kg.read_kv(0, len(prompt) + 2)]
    return out


@pytest.mark.parametrize("head_dim", [64, 128])
def test_contexts_with_different_caches_share_an_arena(head_dim):
    from tests import parity as P
    base = dataclasses.replace(I.SHAPES["small_bf16"], head_dim=head_dim, n_heads=512 // head_dim)
    W = I.gen_weights(base, seed=5, alpha=0.05, head_scale=25.0)
    prompts = [I.gen_prompt(base.vocab, n) for n in (5, 21, 203)]       # decode kernels, short passes, longer ones
    shapes = [dataclasses.replace(base, kv=kv) for kv in ("f16", "bf16", "f32")]
    alone = []
    for s in shapes:
        kg = P.load_model(s, W, 256, kv_page_tokens=32)
        alone.append(_outputs(kg, prompts))
        kg.close()
    first = P.load_model(shapes[0], W, 256, kv_page_tokens=32)
    for s, want in zip(shapes[1:], alone[1:]):
        kg = P.load_model(s, W, 256, kv_page_tokens=32)
        assert kg.weight_bytes == first.weight_bytes
        kg._chk(kg.L.kg_bind(kg.h, first.arena.data_ptr(), first.weight_bytes, kg.kv.data_ptr(), kg.kv_bytes,
                             kg.scratch.data_ptr(), kg.scratch_bytes, kg.stream.cuda_stream))
        kg.load_weights((k, l, W[(k, l)]) for k, l, _, _ in I.tensor_list(s))
        for who, expected in ((kg, want), (first, alone[0])):
            for a, b in zip(_outputs(who, prompts), expected):
                np.testing.assert_array_equal(a, b)
        kg.close()
    first.close()
