"""Kernels that small calls no longer take, on the cases of the tests that small calls used to cover them with."""
import numpy as np
import pytest

import oracle
from moe_inputs import make_logits
from helpers import GATE_ATOL, GATE_RTOL
import test_gpu_permute as permute
from test_gpu_router import _gpu_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["normal", "ties", "dupcols", "zeros", "tiny", "equal", "onehot"])
@pytest.mark.parametrize("E,K", [(8, 2), (64, 8), (64, 6), (7, 3), (16, 1), (4, 4), (100, 5), (48, 4), (90, 33), (1, 1)])
def test_selection_by_lists(kind, E, K):
    """More than 4096 tokens: sorted lists (K <= 8) over 1, 2, 4 or 8 lanes, arg-max rounds beyond."""
    T = 4101
    logits = np.tile(make_logits(103 + E, 300, E, kind), (14, 1))[:T]
    want_idx, want_gate = oracle.topk_gates(logits, K, True)
    _, idx, gate = _gpu_topk(logits, K, True)
    np.testing.assert_array_equal(idx, want_idx)
    np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=GATE_ATOL)


@pytest.mark.parametrize("T,H,E,K,capacity,kind,bf16", [
    (2048, 256, 16, 4, 512, "onehot", True),     # heavy drops on expert 0
    (37, 3072, 12, 5, 0, "normal", True),        # 6 KiB rows
    (90, 24, 256, 64, 0, "normal", False),       # the limits of E and K
    (300, 40, 9, 1, 1, "normal", True),          # capacity 1
    (1, 8, 10, 2, 0, "normal", True),
])
def test_dispatch_in_three_launches(T, H, E, K, capacity, kind, bf16):
    import paper_2504_14960_amd as moe
    moe.set_option("permute_fused", 0)
    try:
        permute.test_permute_maps_and_rows_are_bit_exact(T, H, E, K, capacity, kind, bf16)
    finally:
        moe.set_option("permute_fused", 1)

