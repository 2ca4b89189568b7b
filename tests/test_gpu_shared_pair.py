"""The shared expert's products in one launch with the routed experts': every pair of workgroup widths that the option takes, row counts
at the edges of the narrow kernel's forms, fewer routed rows than tokens, and the same bits for the routed experts as without."""
import pytest

from helpers import assert_close, guard_margins, to_dev, to_host
from moe_inputs import get_config, make_layer_inputs
from test_gpu_layer import oracle_layer

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_afterwards():
    import paper_2504_14960_amd as moe
    yield
    moe.set_option("gemm_pair", -1)
    moe.set_option("gemm_stream", -1)


def _layer(inp, ws_fill=0xFF, capacity=0):
    import torch
    import paper_2504_14960_amd as moe
    c = inp.cfg
    d = {k: to_dev(v) for k, v in inp.tensors.items()}
    bias = None if inp.bias is None else to_dev(inp.bias)
    nbytes = moe.layer_workspace_bytes(c.T, c.H, c.E, c.K, c.F, c.shared_F, capacity, moe.MOE_BF16)
    lay = moe.layer_workspace_layout(c.T, c.H, c.E, c.K, c.F, c.shared_F, capacity, moe.MOE_BF16)
    ws = torch.full((nbytes,), ws_fill, dtype=torch.uint8, device="cuda")      # NaN patterns: nothing unwritten is read
    y = torch.empty_like(d["x"])
    moe.layer_forward(d["x"], d["w_router"], bias, d["w_gate"], d["w_up"], d["w_down"], d["ws_gate"], d["ws_up"], d["ws_down"],
                      c.K, c.renormalize, capacity, y, ws)
    torch.cuda.synchronize()
    rows = int(ws[lay["expert_offsets"]:][:4 * (c.E + 1)].view(torch.int32)[-1])   # kept rows
    y_perm = ws[lay["y_perm"]:lay["y_perm"] + rows * c.H * 2].clone()
    return to_host(y), y_perm


# tokens: up to 16 rows in all, 16 and 17, 32 and 33, 64 and 65, 128 rows of the shared expert; contractions that end inside a
# block, columns inside a workgroup's
@pytest.mark.parametrize("T,H,F,Fs,E,K", [
    (5, 192, 64, 320, 6, 3), (16, 192, 128, 448, 4, 2), (17, 320, 64, 576, 4, 2), (32, 128, 192, 2112, 8, 2), (33, 576, 64, 320, 4, 1),
    (64, 192, 64, 1344, 4, 2), (65, 320, 128, 448, 6, 2), (128, 192, 64, 704, 8, 4)])
def test_pairs_against_the_oracle(T, H, F, Fs, E, K):
    import torch
    import paper_2504_14960_amd as moe
    cfg = get_config("qwen2_57b_a14b").scaled(T=T, H=H, F=F, E=E, K=K, shared_F=Fs, seed=8100 + T)
    inp = make_layer_inputs(cfg)
    guard_margins(inp, K)
    want = oracle_layer(inp, 0)
    moe.set_option("gemm_pair", 0)
    y, y_perm = _layer(inp)
    assert_close(y, want.y, True, "y, one after the other")
    for option in (22, 24, 28, 42, 44, 48, 82, 84, 88, -1):
        moe.set_option("gemm_pair", option)
        got, got_perm = _layer(inp)
        assert_close(got, want.y, True, f"y, pairs {option}")
        assert torch.equal(got_perm, y_perm), option


# With a capacity there may be up to 16 routed rows in all, and more of the shared expert: no pair then, whose workgroups for so few
# rows hold 16 of any expert.  17, 33, 64 and 128 tokens; a pair by default where both products were one; 16 tokens, which stay paired
@pytest.mark.parametrize("T,H,F,Fs,E,K,capacity", [
    (17, 192, 128, 448, 8, 1, 2), (33, 576, 64, 320, 4, 2, 1), (64, 192, 64, 1344, 16, 1, 1), (128, 192, 64, 704, 8, 4, 2),
    (32, 1024, 1024, 2048, 16, 1, 1), (16, 192, 128, 448, 4, 2, 4), (17, 320, 64, 576, 17, 1, 1)])
def test_fewer_routed_rows_than_tokens(T, H, F, Fs, E, K, capacity):
    import torch
    import paper_2504_14960_amd as moe
    cfg = get_config("qwen2_57b_a14b").scaled(T=T, H=H, F=F, E=E, K=K, shared_F=Fs, seed=8300 + T)
    inp = make_layer_inputs(cfg)
    guard_margins(inp, K)
    want = oracle_layer(inp, capacity)
    moe.set_option("gemm_pair", 0)
    y, y_perm = _layer(inp, capacity=capacity)
    assert_close(y, want.y, True, "y, one after the other")
    for option in (-1, 22, 24, 28, 42, 44, 48, 82, 84, 88):
        moe.set_option("gemm_pair", option)
        got, got_perm = _layer(inp, capacity=capacity)
        assert_close(got, want.y, True, f"y, pairs {option}")
        assert torch.equal(got_perm, y_perm), option
