"""The layer in one call, in four stage calls and as the training forward: the same bits, whatever the workspace's size."""
import numpy as np
import pytest

from moe_inputs import get_config, make_layer_inputs
from helpers import to_dev, to_host, values


def _sizes(T, H, E, K, F, Fs, capacity):
    """(bytes of the intermediates alone, bytes asked for)"""
    import paper_2504_14960_amd as moe
    lay = moe.layer_workspace_layout(T, H, E, K, F, Fs, capacity, moe.MOE_BF16)
    up = lambda n: (n + 255) // 256 * 256
    if Fs:
        end = up(lay["shared_y"] + T * H * 2)
    else:
        end = up(lay["y_perm"] + moe.max_rows(T, K, E, capacity) * H * 2) + 256     # and the shared expert's two offsets
    return end, moe.layer_workspace_bytes(T, H, E, K, F, Fs, capacity, moe.MOE_BF16)


# few rows on few experts: the sizes at which splitting a routed expert's contraction would pay
FEW = [(256, 1024, 4, 1, 8192, 0), (20, 2048, 2, 1, 2048, 0), (278, 2816, 4, 1, 16000, 90)]


@pytest.mark.parametrize("T,H,E,K,F,capacity", FEW)
def test_workspace_of_a_layer_without_shared_expert_is_its_intermediates(T, H, E, K, F, capacity):
    end, asked = _sizes(T, H, E, K, F, 0, capacity)
    assert asked == end


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,E,K,F,capacity", FEW[:2])
def test_stage_calls_and_training_forward_give_the_bits_of_the_layer(T, H, E, K, F, capacity):
    import torch
    import paper_2504_14960_amd as moe
    cfg = get_config("mixtral8x22b").scaled(T=T, H=H, E=E, K=K, F=F, seed=8100 + T)
    inp = make_layer_inputs(cfg)
    d = {k: to_dev(v) for k, v in inp.tensors.items()}
    bias = None if inp.bias is None else to_dev(inp.bias)
    r_max = moe.max_rows(T, K, E, capacity)
    bf, i32, f32 = (dict(dtype=t, device="cuda") for t in (torch.bfloat16, torch.int32, torch.float32))
    out = {}
    size = moe.layer_workspace_bytes(T, H, E, K, F, 0, capacity, moe.MOE_BF16)
    for name, nbytes in (("layer", size), ("layer with 64 MiB more", size + (64 << 20))):
        ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device="cuda")
        out[name] = torch.empty((T, H), **bf)
        moe.layer_forward(d["x"], d["w_router"], bias, d["w_gate"], d["w_up"], d["w_down"], None, None, None, K,
                          cfg.renormalize, capacity, out[name], ws)
    out["training"] = torch.empty((T, H), **bf)
    ws, gu = torch.empty(size, dtype=torch.uint8, device="cuda"), torch.empty((r_max, 2 * F), **bf)
    moe.layer_forward_train(d["x"], d["w_router"], bias, d["w_gate"], d["w_up"], d["w_down"], K, cfg.renormalize,
                            capacity, out["training"], gu, ws)
    logits, idx, gate = torch.empty((T, E), **f32), torch.empty((T, K), **i32), torch.empty((T, K), **f32)
    counts, offsets = torch.empty((E,), **i32), torch.empty((E + 1,), **i32)
    roa, aor = torch.empty((T * K,), **i32), torch.empty((r_max,), **i32)
    pws = torch.empty((max(moe.permute_workspace_bytes(T, K, E), 256),), dtype=torch.uint8, device="cuda")
    x_perm, h, y_perm = (torch.empty((r_max, n), **bf) for n in (H, F, H))
    out["stages"] = torch.empty((T, H), **bf)
    moe.router_topk(d["x"], d["w_router"], bias, logits, K, cfg.renormalize, idx, gate)
    moe.permute(d["x"], idx, E, capacity, x_perm, counts, offsets, roa, aor, pws)
    moe.grouped_gemm_swiglu(x_perm, offsets, d["w_gate"], d["w_up"], d["w_down"], h, y_perm)
    moe.unpermute_combine(y_perm, roa, gate, None, out["stages"])
    torch.cuda.synchronize()
    for name, y in out.items():
        assert torch.equal(y.view(torch.int16), out["layer"].view(torch.int16)), f"{name} differs from the layer"


@pytest.mark.gpu
def test_shared_expert_takes_all_the_room_or_none():
    """Two results only, a rounding apart: with the partial sums (also with room to spare) and without (whatever is missing)."""
    import torch
    import paper_2504_14960_amd as moe
    T, H, E, K, F, Fs = 64, 512, 4, 2, 128, 8192       # eight splits of the down projection
    cfg = get_config("qwen2_57b_a14b").scaled(T=T, H=H, F=F, E=E, K=K, shared_F=Fs, seed=8200)
    inp = make_layer_inputs(cfg)
    d = {k: to_dev(v) for k, v in inp.tensors.items()}
    bias = None if inp.bias is None else to_dev(inp.bias)
    end, asked = _sizes(T, H, E, K, F, Fs, 0)
    assert asked > end, "the shape is meant to want partial sums"
    y = {}
    for size in (end, end + (asked - end) // 2, asked - 256, asked, 2 * asked):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
        out = torch.empty_like(d["x"])
        moe.layer_forward(d["x"], d["w_router"], bias, d["w_gate"], d["w_up"], d["w_down"], d["ws_gate"], d["ws_up"],
                          d["ws_down"], K, cfg.renormalize, 0, out, ws)
        torch.cuda.synchronize()
        y[size] = to_host(out)
    for size, got in y.items():
        np.testing.assert_array_equal(got, y[asked if size >= asked else end], err_msg=f"{size} bytes of {asked}")
    # one bf16 rounding of y_perm and one of y, at most a unit in the last place (2^-8) each where a sum straddles a boundary
    assert np.linalg.norm(values(y[asked]) - values(y[end])) <= 2e-3 * np.linalg.norm(values(y[end]))
