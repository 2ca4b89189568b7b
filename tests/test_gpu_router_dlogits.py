"""The softmax Jacobian of the router's backward in both its forms (one wave, one lane per token), against the oracle."""
import numpy as np
import pytest

import oracle
from moe_inputs import make_logits, make_tokens
from helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("renorm", [False, True])
@pytest.mark.parametrize("T,E,K", [
    (5, 64, 8),        # the last lane holds an expert; a ragged last workgroup
    (9, 65, 64),       # two logits per lane, a slot on every lane
    (130, 256, 8),
    (2048, 2, 2),      # the last token count of the wave form for two experts, and the first of the lane form
    (2049, 2, 2),
])
def test_dlogits_against_the_oracle(T, E, K, renorm):
    import torch
    import paper_2504_14960_amd as moe
    rng = np.random.default_rng(E * 100 + T)
    logits = make_logits(9500 + E, T, E, "normal").astype(np.float32)
    idx = oracle.topk_gates(logits, K, renorm)[0].copy()
    if K > 2:
        idx[::3, K - 1] = E          # a slot without an expert
        idx[1::3, 1] = idx[1::3, 0]  # an expert named twice
    dgate = rng.standard_normal((T, K)).astype(np.float32)
    x, w = make_tokens(9501, T, 8, bf16=True), make_tokens(9502, E, 8, bf16=True)
    want = oracle.router_backward(x, w, logits, idx, dgate, renorm)[0]
    dl = torch.full((T, E), float("nan"), dtype=torch.float32, device="cuda")
    moe.router_backward(to_dev(x), to_dev(w), to_dev(logits), to_dev(idx), to_dev(dgate), renorm, dl, None, None, None, None)
    torch.cuda.synchronize()
    # fp32 softmax Jacobian against fp64, as for the whole router's backward
    np.testing.assert_allclose(dl.cpu().numpy(), want, rtol=2e-4, atol=2e-6 * np.abs(dgate).max())
