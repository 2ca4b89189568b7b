"""Large tiles on eight waves where an expert has few rows by R_max and the contraction is short, on four otherwise: the same
bits on both sides of the line, with and without the skip of waves that have no rows, and nothing past the last row."""
import pytest
import torch

import paper_2504_14960_amd as moe

pytestmark = pytest.mark.gpu

BF = dict(dtype=torch.bfloat16, device="cuda")
FEW = [128, 1, 0, 129, 64, 65, 96, 97, 193, 0, 257, 33, 128, 2]           # 85 rows on average, tails that leave waves without rows
MANY_EXPERTS = FEW + [40, 127, 0, 130]                                   # more than 16: the idle waves skip by themselves


@pytest.fixture(autouse=True)
def _large_tiles():
    moe.set_option("gemm_stream", 0)
    yield
    for name in ("gemm_stream", "gemm_idle_skip"):
        moe.set_option(name, -1)
    moe.set_option("gemm_tile_rows", 0)


def _products(R_max, x, off, wg, wu, wd):
    """h and y, h and the pre-activations of the saving form, over R_max rows of which the last ones belong to no expert."""
    E, F, H = wg.shape
    xp = torch.zeros(R_max, H, **BF)
    xp[:x.shape[0]] = x
    h, y, hs, gu = (torch.full((R_max, n), 7.0, **BF) for n in (F, H, F, 2 * F))
    moe.expert_gate_up(xp, off, wg, wu, h)
    moe.expert_down(h, off, wd, y)
    moe.expert_gate_up_saving(xp, off, wg, wu, hs, gu)
    torch.cuda.synchronize()
    for t in (h, y, hs, gu):
        assert bool((t[x.shape[0]:] == 7.0).all()), "rows past the last expert's"
    return [t[:x.shape[0]] for t in (h, y, hs, gu)]


# contractions on both sides of 2048 elements, a ragged last N-tile, two k-tiles
@pytest.mark.parametrize("counts,H,F", [(FEW, 128, 384), (FEW, 2048, 128), (FEW, 2176, 128), (FEW, 384, 2048), (MANY_EXPERTS, 640, 128)])
@pytest.mark.parametrize("rows,skip", [(0, -1), (128, 0), (128, 1), (192, 1), (256, 1)])
def test_same_bits_on_four_and_eight_waves(counts, H, F, rows, skip):
    E = len(counts)
    off = torch.zeros(E + 1, dtype=torch.int32)
    off[1:] = torch.tensor(counts).cumsum(0)
    R = int(off[-1])
    gen = torch.Generator(device="cuda").manual_seed(H + F)
    x, wg, wu, wd = (torch.empty(s, **BF).normal_(0.0, std, generator=gen)
                     for s, std in (((R, H), 1.0), ((E, F, H), 0.02), ((E, F, H), 0.02), ((E, H, F), 0.02)))
    moe.set_option("gemm_tile_rows", rows)
    moe.set_option("gemm_idle_skip", skip)
    off = off.cuda()
    want = None
    lines = {n * E // K for n in (220000, 440000) for K in (H, F)}           # of the plain products and of the one that saves
    for R_max in sorted({R} | {line + d for line in lines for d in (0, 1) if line >= R}):
        got = _products(R_max, x, off, wg, wu, wd)
        want = want or got
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16)), R_max
    ref = torch.cat([x[off[e]:off[e + 1]].float() @ wg[e].float().T for e in range(E)])
    gate = want[3][:, :F].float()
    # both sums in fp32, ours rounded once: half a bf16 step of the value, and the sums' noise (1e-5 of the largest)
    assert bool(((gate - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max()).all())
