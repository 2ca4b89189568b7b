"""The router, dispatch and combine kernels that small batches take, against the oracle."""
import numpy as np
import pytest

import oracle
from moe_inputs import get_config, make_layer_inputs
from helpers import GATE_RTOL, LOGIT_ATOL, guard_margins
from test_gpu_router import _gpu_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,E,K,bias,renorm", [
    (1, 4096, 8, 2, None, True),            # one token, one block of experts
    (17, 40, 17, 3, "normal", True),        # a step that is mostly past the row; one expert in the second block
    (777, 1032, 64, 8, None, False),        # tokens past the last block repeat the last one
    (1024, 136, 128, 6, "normal", True),    # 32 tokens per workgroup; two logits per lane in the selection
    (2048, 1032, 100, 9, None, True),       # more slots than the list form takes
])
def test_experts_spread_over_workgroups(T, H, E, K, bias, renorm):
    import paper_2504_14960_amd as moe
    cfg = get_config("mixtral8x7b").scaled(T=T, H=H, E=E, K=K, bias=bias, seed=3100 + E)
    inp = make_layer_inputs(cfg, ["x", "w_router", "bias"])
    guard_margins(inp, K)
    l64 = oracle.router_logits(inp["x"], inp["w_router"], inp.bias)
    want_idx, want_gate = oracle.topk_gates(l64.astype(np.float32), K, renorm)
    moe.set_option("router_tile", 8)
    try:
        logits, idx, gate = _gpu_topk(np.zeros((T, E), np.float32), K, renorm, inp["x"], inp["w_router"], inp.bias)
    finally:
        moe.set_option("router_tile", 0)
    assert np.abs(logits - l64).max() <= LOGIT_ATOL
    np.testing.assert_array_equal(idx, want_idx)
    np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=2e-5)   # a softmax moves by at most delta / 4


@pytest.mark.parametrize("kind", ["ties", "all_equal", "subnormal"])
@pytest.mark.parametrize("T,E,K", [(3, 64, 64), (5, 63, 8), (4, 128, 5), (4096, 65, 2), (4097, 65, 2)])
def test_selection_by_rank(kind, T, E, K):
    """Exact against the oracle on the same logits, at both ends of the lanes and on both sides of the token limit."""
    rng = np.random.default_rng(E * 7 + K)
    logits = rng.standard_normal((T, E)).astype(np.float32)
    if kind == "ties":
        logits = np.round(logits * 2) / 2
        logits[:, ::3] = -0.0
    elif kind == "all_equal":
        logits[:] = 1.25
    else:
        logits *= np.float32(1e-41)
    want_idx, want_gate = oracle.topk_gates(logits, K, False)
    _, idx, gate = _gpu_topk(logits, K, False)
    np.testing.assert_array_equal(idx, want_idx)
    np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=1e-6)
