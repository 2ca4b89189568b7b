"""Large tiles whose lower waves have no rows: those waves skip all k-tiles but the last, and multiply that one with whatever
their registers hold.  Nothing of it may reach the outputs or the largest |h|: the bits of the kernels without the skip."""
import pytest
import torch

import paper_2504_14960_amd as moe

pytestmark = pytest.mark.gpu

# full tiles, tails that leave the lower waves of each tile height without rows (up to 128, 96 and 64 rows), one row, none
COUNTS = [256, 1, 0, 128, 129, 96, 97, 64, 65, 300, 192, 193, 0, 257, 33, 512, 130, 2]


def _both(run, rows):
    moe.set_option("gemm_stream", 0)
    moe.set_option("gemm_tile_rows", rows)
    out = []
    try:
        for skip in (0, 1):
            moe.set_option("gemm_idle_skip", skip)
            out.append(run())
            torch.cuda.synchronize()
    finally:
        moe.set_option("gemm_idle_skip", -1)
        moe.set_option("gemm_tile_rows", 0)
        moe.set_option("gemm_stream", -1)
    for plain, skipped in zip(*out):
        assert torch.equal(plain.view(torch.uint8), skipped.view(torch.uint8))


def _offsets():
    o = torch.zeros(len(COUNTS) + 1, dtype=torch.int32)
    o[1:] = torch.tensor(COUNTS).cumsum(0)
    return o.cuda(), int(o[-1])


@pytest.mark.parametrize("rows", [256, 192, 128])
@pytest.mark.parametrize("H,F", [(256, 384), (384, 256)])      # two and three k-tiles of 128 bytes in FP8, four and six in bf16
def test_waves_without_rows_leave_no_trace(H, F, rows):
    off, R = _offsets()
    E = len(COUNTS)
    gen = torch.Generator(device="cuda").manual_seed(H)

    def draw(*shape):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)

    def codes(*shape):
        c = torch.empty(shape, dtype=torch.uint8, device="cuda")
        moe.fp8_quantize(draw(*shape), 448 / 5.5, c)
        return c

    x, wg, wu, wd = draw(R, H), draw(E, F, H), draw(E, F, H), draw(E, H, F)

    def bf16():
        h, y = torch.zeros(R, F, dtype=torch.bfloat16, device="cuda"), torch.zeros_like(x)
        moe.expert_gate_up(x, off, wg, wu, h)
        moe.expert_down(h, off, wd, y)
        return h, y

    _both(bf16, rows)
    x8, wg8, wu8, wd8 = codes(R, H), codes(E, F, H), codes(E, F, H), codes(E, H, F)

    def fp8():
        h, y = torch.zeros(R, F, dtype=torch.uint8, device="cuda"), torch.zeros_like(x)
        amax = torch.zeros(1, device="cuda")
        moe.expert_gate_up_fp8(x8, off, wg8, wu8, 1e-4, 1e-4, 64.0, h, amax)
        moe.expert_down_fp8(h, off, wd8, 1e-4, y)
        assert bool(torch.isfinite(amax).all()) and float(amax) > 0
        return h, y, amax

    _both(fp8, rows)


@pytest.mark.parametrize("rows", [256, 192, 128])
@pytest.mark.parametrize("H,F", [(256, 384), (384, 256)])
def test_waves_without_rows_in_fp8_with_three_activation_stages(H, F, rows):
    off, R = _offsets()
    E = len(COUNTS)
    gen = torch.Generator(device="cuda").manual_seed(H + 1)

    def codes(*shape):
        c = torch.empty(shape, dtype=torch.uint8, device="cuda")
        moe.fp8_quantize(torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen), 448 / 5.5, c)
        return c

    x8, wg8, wu8, wd8 = codes(R, H), codes(E, F, H), codes(E, F, H), codes(E, H, F)

    def fp8():
        h, y = torch.zeros(R, F, dtype=torch.uint8, device="cuda"), torch.zeros(R, H, dtype=torch.bfloat16, device="cuda")
        amax = torch.zeros(1, device="cuda")
        moe.expert_gate_up_fp8(x8, off, wg8, wu8, 1e-4, 1e-4, 64.0, h, amax)
        moe.expert_down_fp8(h, off, wd8, 1e-4, y)
        assert bool(torch.isfinite(amax).all()) and float(amax) > 0
        return h, y, amax

    moe.set_option("fp8_deep_weights", 0)
    try:
        _both(fp8, rows)
    finally:
        moe.set_option("fp8_deep_weights", 1)
