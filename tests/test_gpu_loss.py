"""Eq. 3's row losses and its gradient's sums over vocabularies that a block keeps in registers and larger ones."""
import numpy as np
import pytest

from paper_2404_18911_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 1008, 4096, 4112, 32768, 32784])
def test_row_losses_match_the_logits_they_are_taken_from(V):
    """The losses against float64 from the very draft logits the step used, and sum_v (q - p) = 0 through the own head's
    gradient: its rows sum to zero over the vocabulary.  Float32 exponentials and sums: 1e-5 of a row's loss."""
    import torch
    from paper_2404_18911_amd import binding as B
    from tests import parity as P
    shape = I.ModelShape("loss", 1, 128, 2, 64, 256, V, 1, "f32", adapter=I.ADAPTER_ATTN_HEAD)
    W = I.gen_weights(shape, seed=3, alpha=1.0, head_scale=10.0)
    n = 5
    kg = P.load_model(shape, W, 64, kv_page_tokens=16)
    kg.train_bind(n)
    g = torch.Generator(device="cuda").manual_seed(V)
    F = torch.randn(n, 128, generator=g, device="cuda")
    Zt = 2.0 * torch.randn(n, V, generator=g, device="cuda")
    Zt[0, 0] = 30.0
    loss = kg.train_accumulate_features(F, Zt)
    Z = torch.from_numpy(kg.train_read(B.TRAIN_DRAFT_LOGITS, n)).double()
    rows = kg.train_read(B.TRAIN_ROW_LOSSES, n).astype(np.float64)
    want = -(torch.softmax(Zt.cpu().double(), -1) * torch.log_softmax(Z, -1)).sum(-1).numpy()
    np.testing.assert_allclose(rows, want, rtol=1e-5)
    assert abs(loss - want.sum()) <= 1e-5 * want.sum()
    head = B.split_param_block(kg.train_read(B.TRAIN_GRADIENTS, n), shape)["head"].astype(np.float64)
    assert np.all(np.abs(head.sum(0)) <= 1e-5 * np.abs(head).sum(0) + 1e-6)
    kg.close()
