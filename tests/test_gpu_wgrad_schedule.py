"""Weight gradients of more tiles than a workgroup works out at a time (64), with several experts to a lane and empty ones
between them: every tile is written, at its place, with the bits that one tile per workgroup gives."""
import numpy as np
import pytest
import torch

import paper_2504_14960_amd as moe

pytestmark = pytest.mark.gpu

BF = dict(dtype=torch.bfloat16, device="cuda")


def _gradients(E, H, F, counts, workgroups):
    gen = torch.Generator(device="cuda").manual_seed(E + H)
    offsets = torch.zeros(E + 1, dtype=torch.int32)
    offsets[1:] = torch.from_numpy(counts).cumsum(0)
    R = int(offsets[-1])

    def draw(*shape):
        return torch.empty(shape, **BF).normal_(generator=gen)

    x, dy, h, gu = draw(R, H), draw(R, H), draw(R, F), draw(R, 2 * F)
    wg, wu, wgu_t, wd_t = draw(E, F, H), draw(E, F, H), draw(E, H, 2 * F), draw(E, F, H)
    dx = torch.empty(R, H, **BF)
    dw = [torch.full(s, 7.0, **BF) for s in ((E, F, H), (E, F, H), (E, H, F))]
    ws = torch.empty(moe.expert_backward_workspace_bytes(R, H, F, E) + 256, dtype=torch.uint8, device="cuda")
    moe.set_option("gemm_workgroups", workgroups)
    try:
        moe.grouped_gemm_swiglu_backward(x, h, gu, dy, offsets.cuda(), wg, wu, wgu_t, wd_t, dx, *dw, ws)
        torch.cuda.synchronize()
    finally:
        moe.set_option("gemm_workgroups", 0)
    return dw, dy, h, offsets.tolist()


@pytest.mark.parametrize("E,H,F", [(150, 384, 256), (256, 128, 128), (9, 2304, 2048)])
def test_more_tiles_than_are_worked_out_at_a_time(E, H, F):
    rng = np.random.default_rng(E)
    counts = rng.integers(0, 70, size=E)
    counts[rng.integers(0, E, size=E // 4)] = 0            # empty experts, next to one another too
    counts[-1] = 0
    one, dy, h, off = _gradients(E, H, F, counts, 0)       # as many workgroups as there are tiles, at most one per compute unit
    few, _, _, _ = _gradients(E, H, F, counts, 8)          # one per XCD
    for a, b in zip(one, few):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        want = dy[off[e]:off[e + 1]].float().T @ h[off[e]:off[e + 1]].float()
        # products and sums in fp32 on both sides, the result rounded once: half a bf16 step of the largest, and the sums' noise
        assert (few[2][e].float() - want).abs().max() <= 2.0 ** -8 * max(want.abs().max().item(), 1e-30) * 1.01, f"expert {e}"


@pytest.mark.parametrize("E,H,F", [(1, 128, 128), (4, 1024, 1024), (3, 384, 640), (8, 1024, 1024), (5, 896, 1152)])
def test_few_tiles_are_128_rows_high(E, H, F):
    """Launches whose 256-row tiles would leave half of the workgroups without one: the bits of the 256-row tiles, which eight
    workgroups get, with many rows and few, and experts without rows."""
    rng = np.random.default_rng(E * H)
    counts = rng.integers(1, 900, size=E)
    if E > 2:
        counts[1], counts[E // 2] = 0, 3
    low, dy, h, off = _gradients(E, H, F, counts, 0)
    tall, _, _, _ = _gradients(E, H, F, counts, 8)
    for a, b in zip(low, tall):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        want = dy[off[e]:off[e + 1]].float().T @ h[off[e]:off[e + 1]].float()
        assert (low[2][e].float() - want).abs().max() <= 2.0 ** -8 * max(want.abs().max().item(), 1e-30) * 1.01, f"expert {e}"
