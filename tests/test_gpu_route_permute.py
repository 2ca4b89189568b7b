"""Routing and dispatch of a handful of tokens in one launch: what it leaves in the layer's workspace and the layer's output have
the bits of the separate launches (the same dispatch option off)."""
import pytest

pytestmark = pytest.mark.gpu

# (H, E, K): one piece of a row, one expert, every expert chosen, 16 experts (64 assignments), a row of 16 KiB, a part of one
SHAPES = [(8, 1, 1), (8, 16, 3), (200, 3, 3), (1600, 16, 16), (4096, 8, 2), (8192, 4, 2), (8184, 7, 5)]


@pytest.fixture(autouse=True)
def _default_afterwards():
    import paper_2504_14960_amd as moe
    yield
    moe.set_option("permute_fused", 1)


def _layer(T, H, E, K, capacity, renorm, shared, fused, special=False):
    import torch
    import paper_2504_14960_amd as moe
    gen = torch.Generator(device="cuda").manual_seed(100 * H + 10 * E + T)
    F, Fs = 64, 128 if shared else 0

    def make(*shape, std=0.05):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    x, wr, bias = make(T, H, std=1.0), make(E, H), torch.randn(E, generator=gen, device="cuda")
    if special:                       # a token without finite logits, and equal logits for all experts of another
        x[0, 0] = float("nan")
        wr[:] = wr[:1].clone()
        bias.zero_()
    w = [make(E, F, H), make(E, F, H), make(E, H, F)]
    s = [make(Fs, H), make(Fs, H), make(H, Fs)] if shared else [None] * 3
    ws = torch.full((moe.layer_workspace_bytes(T, H, E, K, F, Fs, capacity, moe.MOE_BF16),), 0x5A, dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    moe.set_option("permute_fused", fused)
    moe.layer_forward(x, wr, bias, *w, *s, K, renorm, capacity, y, ws)
    at = moe.layer_workspace_layout(T, H, E, K, F, Fs, capacity, moe.MOE_BF16)
    rows = moe.max_rows(T, K, E, capacity)
    size = dict(logits=T * E * 4, topk_idx=T * K * 4, topk_gate=T * K * 4, expert_counts=E * 4, expert_offsets=(E + 1) * 4,
                row_of_assign=T * K * 4, assign_of_row=rows * 4)
    got = {n: ws[at[n]:at[n] + size[n]].clone() for n in size}
    kept = int(got["expert_offsets"].view(torch.int32)[E])
    got["x_perm"] = ws[at["x_perm"]:at["x_perm"] + kept * H * 2].clone()   # rows past the kept ones are nobody's
    got["y"] = y.view(torch.int16)
    return got


@pytest.mark.parametrize("capacity", [0, 1])
@pytest.mark.parametrize("H,E,K", SHAPES)
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5])
def test_bits_of_the_separate_launches(T, H, E, K, capacity):
    import torch
    one = _layer(T, H, E, K, capacity, T % 2 == 0, False, 1)
    apart = _layer(T, H, E, K, capacity, T % 2 == 0, False, 0)
    for name in apart:
        assert torch.equal(one[name], apart[name]), name


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("T", [1, 4])
def test_with_a_shared_expert_ties_and_nan(T, special):
    import torch
    one, apart = (_layer(T, 256, 8, 2, 0, True, True, fused, special) for fused in (1, 0))
    for name in apart:
        assert torch.equal(one[name], apart[name]), name
