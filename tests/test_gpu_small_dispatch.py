"""The router, dispatch and combine kernels that small batches take, against the oracle."""
import numpy as np
import pytest

import oracle
from moe_inputs import get_config, make_layer_inputs, make_tokens
from helpers import GATE_RTOL, LOGIT_ATOL, assert_close, guard_margins, to_dev, values
from test_gpu_permute import _gpu_combine, _gpu_permute, _idx
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


@pytest.mark.parametrize("T,H,E,K,bias,renorm", [
    (1, 4096, 8, 2, None, True),            # one token
    (3, 40, 1, 1, None, False),             # one expert; a step that is mostly past the row
    (255, 264, 5, 5, "normal", True),       # every expert selected
    (513, 1032, 12, 3, None, False),        # four tokens per workgroup, one of them in the last
    (1023, 136, 16, 4, "normal", True),     # sixteen experts, no padding
    (2048, 72, 15, 9, None, True),          # eight tokens per workgroup
    (3001, 264, 16, 8, None, True),         # sixteen, nine of them in the last
    (4096, 64, 3, 2, "normal", False),      # the most tokens
])
def test_router_and_selection_of_up_to_16_experts_in_one_launch(T, H, E, K, bias, renorm):
    cfg = get_config("mixtral8x7b").scaled(T=T, H=H, E=E, K=K, bias=bias, seed=3200 + E)
    inp = make_layer_inputs(cfg, ["x", "w_router", "bias"])
    guard_margins(inp, K)
    l64 = oracle.router_logits(inp["x"], inp["w_router"], inp.bias)
    logits, idx, gate = _gpu_topk(np.zeros((T, E), np.float32), K, renorm, inp["x"], inp["w_router"], inp.bias)
    assert np.abs(logits - l64).max() <= LOGIT_ATOL
    want_idx, want_gate = oracle.topk_gates(logits, K, renorm)     # the selection on the kernel's own logits
    np.testing.assert_array_equal(idx, want_idx)
    np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=1e-6)
    if E > 1:                                                      # equal weight rows: exact ties, lower index first
        w = inp["w_router"].copy()
        w[1::2] = w[0]
        logits, idx, gate = _gpu_topk(np.zeros((T, E), np.float32), K, renorm, inp["x"], w, None)
        want_idx, want_gate = oracle.topk_gates(logits, K, renorm)
        np.testing.assert_array_equal(idx, want_idx)
        np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=1e-6)


@pytest.mark.parametrize("T,H,E", [(64, 4096, 16), (65, 4096, 16), (1, 6376, 9), (5, 8192, 8), (512, 4096, 16), (513, 4104, 16)])
def test_both_sides_of_the_one_launch_line(T, H, E):
    """One launch or two: the same sums in the same order, so the same bits."""
    import paper_2504_14960_amd as moe
    cfg = get_config("mixtral8x7b").scaled(T=T, H=H, E=E, K=3, bias="normal", seed=3250 + T)
    inp = make_layer_inputs(cfg, ["x", "w_router", "bias"])
    runs = []
    for tile in (0, 8):
        moe.set_option("router_tile", tile)
        try:
            runs.append(_gpu_topk(np.zeros((T, E), np.float32), 3, True, inp["x"], inp["w_router"], inp.bias))
        finally:
            moe.set_option("router_tile", 0)
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("T,H,E,K,bias,renorm", [
    (5, 64, 17, 2, None, True),             # 32 x 32, one stage; fewer tokens than a tile, the selection in the workgroup
    (300, 512, 32, 4, "normal", False),     # as many stages as the ring
    (333, 704, 33, 3, None, True),          # two expert blocks, one expert in the second; three stages past the ring
    (4164, 1280, 64, 6, "normal", True),    # 32 x 64
    (2300, 2048, 128, 9, None, False),      # 32 x 64, two blocks, more slots than the list form takes
    (20000, 576, 40, 4, "normal", True),    # 64 x 64, a ragged last tile
    (8100, 512, 100, 8, "normal", False),   # 64 x 64, two blocks, a ragged last tile
    (9500, 3072, 100, 8, None, True),       # 128 x 64, two blocks, several stages past the ring
    (8200, 640, 128, 9, None, False),       # 128 x 64, two blocks
    (17000, 4096, 64, 6, "normal", True),   # 128 x 64, the selection in the workgroup
])
def test_router_tiles_of_tokens_and_experts(T, H, E, K, bias, renorm):
    import paper_2504_14960_amd as moe
    cfg = get_config("mixtral8x7b").scaled(T=T, H=H, E=E, K=K, bias=bias, seed=3300 + E)
    inp = make_layer_inputs(cfg, ["x", "w_router", "bias"])
    l64 = oracle.router_logits(inp["x"], inp["w_router"], inp.bias)
    moe.set_option("router_tile", 16)
    try:
        logits, idx, gate = _gpu_topk(np.zeros((T, E), np.float32), K, renorm, inp["x"], inp["w_router"], inp.bias)
    finally:
        moe.set_option("router_tile", 0)
    assert np.abs(logits - l64).max() <= LOGIT_ATOL
    want_idx, want_gate = oracle.topk_gates(logits, K, renorm)     # the selection on the kernel's own logits
    np.testing.assert_array_equal(idx, want_idx)
    np.testing.assert_allclose(gate, want_gate, rtol=GATE_RTOL, atol=1e-6)


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


@pytest.mark.parametrize("T,H,E,K,capacity,kind,bf16", [
    (1, 4096, 8, 2, 0, "normal", True),           # one workgroup, three of its four tokens missing
    (1023, 24, 64, 8, 0, "normal", True),         # rows of 48 bytes: most waves hold no piece
    (1024, 2056, 12, 3, 100, "onehot", True),     # five pieces of a KiB over four waves; drops
    (1025, 1544, 256, 2, 0, "normal", False),     # 16 tokens per workgroup, 6 KiB rows, every lane of the scan
    (2000, 2560, 100, 4, 64, "normal", False),    # 10 KiB rows
    (1100, 8192, 9, 1, 0, "normal", True),        # 16 KiB rows, the largest
    (90, 8, 64, 64, 0, "normal", True),           # 4 workgroups' worth of 64-assignment units per token group
])
def test_one_launch_dispatch_with_histograms(T, H, E, K, capacity, kind, bf16):
    import paper_2504_14960_amd as moe
    idx = _idx(4100 + T, T, E, K, kind)[0].copy()
    idx[T // 2, 0] = E           # an index outside [0, E): a dropped assignment
    x = make_tokens(4101, T, H, bf16=bf16)
    want = oracle.permute(x, idx, E, capacity)
    moe.set_option("permute_fused", 4)
    try:
        x_perm, counts, offsets, roa, aor = _gpu_permute(x, idx, E, capacity)
        maps_only = _gpu_permute(None, idx, E, capacity)
    finally:
        moe.set_option("permute_fused", 1)
    for got in ((counts, offsets, roa, aor), maps_only[1:]):
        for a, b in zip(got, (want.counts, want.offsets, want.row_of_assign, want.assign_of_row)):
            np.testing.assert_array_equal(a, b)
    np.testing.assert_array_equal(x_perm[:want.R], want.x_perm[:want.R])
    assert (x_perm[want.R:] == 0).all(), "rows past the kept total must be left untouched"


@pytest.mark.parametrize("T,H,E,K,capacity", [(1, 4096, 8, 2, 0), (37, 1032, 64, 8, 0), (1024, 520, 20, 2, 60), (1500, 2048, 60, 4, 0)])
def test_one_launch_fp8_dispatch_with_histograms(T, H, E, K, capacity):
    import torch
    import paper_2504_14960_amd as moe
    idx = _idx(4300 + T, T, E, K, "onehot" if capacity else "normal")[0]
    x = make_tokens(4301, T, H, bf16=True)
    r_max = moe.max_rows(T, K, E, capacity)
    i32 = dict(dtype=torch.int32, device="cuda")
    out = []
    for fused in (0, 4):
        xq = torch.full((r_max + 2, H), 0xAA, dtype=torch.uint8, device="cuda")
        maps = [torch.empty((n,), **i32) for n in (E, E + 1, T * K, r_max)]
        ws = torch.empty((moe.permute_workspace_bytes(T, K, E) + 256,), dtype=torch.uint8, device="cuda")
        amax = torch.zeros(1, dtype=torch.float32, device="cuda")
        moe.set_option("permute_fused", fused)
        try:
            moe.permute_fp8(to_dev(x), to_dev(idx), E, capacity, 23.7, xq[:r_max], *maps, amax, ws)
            torch.cuda.synchronize()
        finally:
            moe.set_option("permute_fused", 1)
        out.append([xq, *maps, amax])
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T,one_launch", [(8192, True), (8193, False)])
def test_many_tokens_of_one_expert_each_leave_the_one_launch_form(T, one_launch):
    """The three-launch form keeps its histograms in the workspace, the one-launch form does not touch it."""
    import torch
    import paper_2504_14960_amd as moe
    H, E, K = 64, 16, 1
    idx = _idx(4500 + T, T, E, K, "normal")[0]
    x = make_tokens(4501, T, H, bf16=True)
    want = oracle.permute(x, idx, E, 0)
    maps = [torch.empty((n,), dtype=torch.int32, device="cuda") for n in (E, E + 1, T, T)]
    ws = torch.full((moe.permute_workspace_bytes(T, K, E) + 256,), 0xAA, dtype=torch.uint8, device="cuda")
    moe.permute(to_dev(x), to_dev(idx), E, 0, torch.empty((T, H), dtype=torch.bfloat16, device="cuda"), *maps, ws)
    torch.cuda.synchronize()
    for got, ref in zip(maps, (want.counts, want.offsets, want.row_of_assign, want.assign_of_row)):
        np.testing.assert_array_equal(got.cpu().numpy(), ref)
    assert bool((ws == 0xAA).all()) == one_launch


@pytest.mark.parametrize("T,H,K,bf16,with_addend", [
    (1, 4104, 2, True, True),          # three slices of a row, the last of 16 bytes
    (3, 3584, 8, True, True),
    (64, 1028, 4, False, True),
    (2047, 1032, 1, True, False),      # the last token count that is split, two slices
    (5, 2056, 20, True, True),         # more than eight slots: the general kernel
])
def test_combine_of_few_tokens(T, H, K, bf16, with_addend):
    rng = np.random.default_rng(T + H)
    rows = T * K + 3
    y_perm = make_tokens(4400, rows, H, bf16=bf16)
    addend = make_tokens(4401, T, H, bf16=bf16) if with_addend else None
    roa = rng.permutation(rows)[:T * K].astype(np.int32)
    roa[::5] = -1
    gate = rng.random((T, K)).astype(np.float32)
    want = oracle.combine(values(y_perm), roa, gate.astype(np.float64), None if addend is None else values(addend))
    got = _gpu_combine(y_perm, roa, gate, addend, T, K)
    assert_close(got, want, bf16, "y")
