"""The weights' transposes, bit for bit: in tiles of 128 x 128, and, with results of more than 140 MiB, of 256 rows x 64 columns, also
where the rows do not divide into tiles.  (The columns always do: the entry point takes multiples of 128.)"""
import pytest
import torch

import paper_2504_14960_amd as moe

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,H,F", [(1, 128, 128), (3, 384, 128), (2, 128, 640), (2, 640, 896), (1, 256, 2048),
                                   (42, 640, 896), (43, 640, 896),      # results on both sides of 140 MiB
                                   (33, 2304, 384), (256, 384, 256)])
def test_weights_transposed_bit_for_bit(E, H, F):
    gen = torch.Generator(device="cuda").manual_seed(E * H + F)

    def draw(*shape):
        return torch.randint(-32768, 32768, shape, dtype=torch.int16, device="cuda", generator=gen)

    wg, wu, wd = draw(E, F, H), draw(E, F, H), draw(E, H, F)
    wgu_t, wd_t = draw(E, H, 2 * F), draw(E, F, H)
    moe.expert_weights_transpose(*(t.view(torch.bfloat16) for t in (wg, wu, wd, wgu_t, wd_t)))
    assert torch.equal(wgu_t[:, :, :F], wg.transpose(1, 2))
    assert torch.equal(wgu_t[:, :, F:], wu.transpose(1, 2))
    assert torch.equal(wd_t, wd.transpose(1, 2))
