"""Schedules of the weight gradients.  More tiles than a workgroup works out at a time (64): several experts to a lane and empty
ones between them; several tiles of an expert and tiles of different lengths on both sides of the 64th.  Every tile is written, at
its place, with the bits that other numbers of workgroups give.  And tiles of 128 rows, where there are few."""
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
    return dw, (x, dy, h, gu, wd_t), offsets.tolist()


@pytest.mark.parametrize("E,H,F", [(150, 384, 256), (256, 128, 128), (9, 2304, 2048)])
def test_more_tiles_than_are_worked_out_at_a_time(E, H, F):
    rng = np.random.default_rng(E)
    counts = rng.integers(0, 70, size=E)
    counts[rng.integers(0, E, size=E // 4)] = 0            # empty experts, next to one another too
    counts[-1] = 0
    one, (_, dy, h, _, _), off = _gradients(E, H, F, counts, 0)   # as many workgroups as there are tiles, at most one per compute unit
    few, _, _ = _gradients(E, H, F, counts, 8)                    # one per XCD
    for a, b in zip(one, few):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        want = dy[off[e]:off[e + 1]].float().T @ h[off[e]:off[e + 1]].float()
        # products and sums in fp32 on both sides, the result rounded once: half a bf16 step of the largest, and the sums' noise
        assert (few[2][e].float() - want).abs().max() <= 2.0 ** -8 * max(want.abs().max().item(), 1e-30) * 1.01, f"expert {e}"


def _fewest_tiles(M, N, experts):
    """256-row tiles of the workgroup that has least of them, eight workgroups, one per XCD: an eighth of every expert's each."""
    per_expert = -(-M // 256) * -(-N // 256)
    return experts * min((x + 1) * per_expert // 8 - x * per_expert // 8 for x in range(8))


# 9 and 3 or 4 tiles of an expert to a workgroup, M-groups of eight and the M-tiles left over; two to seven k-tiles, and nine to
# twelve (640 padded rows per expert on average lie between the two)
@pytest.mark.parametrize("E,H,F,rows", [(26, 2304, 2048, (1, 70, 130, 200, 400, 0)), (28, 1536, 1280, (520, 700, 560, 750, 600, 0))])
def test_tiles_of_several_lengths_on_both_sides_of_the_64th(E, H, F, rows):
    counts = np.array([rows[(e * e + e // 4) % len(rows)] for e in range(E)])
    assert min(_fewest_tiles(H, F, (counts > 0).sum()), _fewest_tiles(F, H, (counts > 0).sum())) > 64
    padded = counts.sum() + 127 * E
    assert (padded <= 640 * E) == (max(rows) < 500)
    few, (x, dy, h, gu, wd_t), off = _gradients(E, H, F, counts, 8)
    one, _, _ = _gradients(E, H, F, counts, 0)
    for a, b in zip(one, few):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        r = slice(off[e], off[e + 1])
        g, u = gu[r].float().split(F, dim=1)
        dh = (dy[r].float() @ wd_t[e].float().T).bfloat16().float()      # rounded before the derivative, as the library does
        sig = torch.sigmoid(g)
        dg, du = (dh * u * sig * (1 + g * (1 - sig))).bfloat16().float(), (dh * g * sig).bfloat16().float()
        for got, left, right, steps in ((few[0], dg, x[r].float(), 4), (few[1], du, x[r].float(), 4), (few[2], dy[r].float(), h[r].float(), 0)):
            want = left.T @ right
            # the result rounded once (as above); and an element of dg or du that falls on the neighbouring bf16 step, through
            # dh's rounding or its own, moves a sum by up to 2^-7 of its product: four of those
            moved = 0.0 if off[e] == off[e + 1] else steps * 2.0 ** -7 * (left.abs().max() * right.abs().max()).item()
            assert (got[e].float() - want).abs().max() <= 2.0 ** -8 * want.abs().max() + moved, f"expert {e}"


@pytest.mark.parametrize("E,H,F", [(1, 128, 128), (4, 1024, 1024), (3, 384, 640), (8, 1024, 1024), (5, 896, 1152)])
def test_few_tiles_are_128_rows_high(E, H, F):
    """Launches whose 256-row tiles would leave half of the workgroups without one: the bits of the 256-row tiles, which eight
    workgroups get, with many rows and few, and experts without rows."""
    rng = np.random.default_rng(E * H)
    counts = rng.integers(1, 900, size=E)
    if E > 2:
        counts[1], counts[E // 2] = 0, 3
    low, (_, dy, h, _, _), off = _gradients(E, H, F, counts, 0)
    tall, _, _ = _gradients(E, H, F, counts, 8)
    for a, b in zip(low, tall):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        want = dy[off[e]:off[e + 1]].float().T @ h[off[e]:off[e + 1]].float()
        assert (low[2][e].float() - want).abs().max() <= 2.0 ** -8 * max(want.abs().max().item(), 1e-30) * 1.01, f"expert {e}"


# one expert and 64, M- and N-tiles that end inside a tile of 128 x 256, several tiles to a workgroup and less than one, up to 97 rows
@pytest.mark.parametrize("E,H,F,most", [(1, 128, 128, 97), (3, 384, 640, 150), (17, 896, 1152, 190), (64, 256, 384, 170), (64, 1024, 896, 120)])
def test_gradients_of_few_rows(E, H, F, most):
    """On eight waves: what eight workgroups and one per compute unit write are the same bits, and right."""
    rng = np.random.default_rng(E + H)
    counts = rng.integers(1, most + 1, size=E)
    if E > 2:
        counts[1], counts[E // 2], counts[-1] = 0, 1, 0
    assert (counts.sum() + 127 * min(E, counts.sum()) + 63) // 64 * 64 <= 224 * E
    few, (x, dy, h, gu, wd_t), off = _gradients(E, H, F, counts, 8)
    one, _, _ = _gradients(E, H, F, counts, 0)
    for a, b in zip(one, few):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    for e in range(E):
        r = slice(off[e], off[e + 1])
        if counts[e] == 0:
            assert not any(t[e].any() for t in few), f"expert {e}"
            continue
        want = dy[r].float().T @ h[r].float()
        assert (few[2][e].float() - want).abs().max() <= 2.0 ** -8 * max(want.abs().max().item(), 1e-30) * 1.01, f"expert {e}"
        g, u = gu[r].float().split(F, dim=1)
        dh = (dy[r].float() @ wd_t[e].float().T).bfloat16().float()
        sig = torch.sigmoid(g)
        du = (dh * g * sig).bfloat16().float()
        want = du.T @ x[r].float()
        # the result rounded once, and four products of an element of du on the neighbouring step, as above
        moved = 4 * 2.0 ** -7 * (du.abs().max() * x[r].abs().max()).item()
        assert (few[1][e].float() - want).abs().max() <= 2.0 ** -8 * want.abs().max() + moved, f"expert {e}"
