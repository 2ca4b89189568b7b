"""The small tiles of the expert products in bf16 and FP8, every form: row counts around the edges of the tiles, columns and
contractions that end inside a tile, a block, a step or a group's share, and the forms that store pre-activations."""
import numpy as np
import pytest

from helpers import assert_close, to_dev, to_host, values
from test_gpu_experts import _case as bf16_case, _run as bf16_run
from test_gpu_fp8 import _case as fp8_case
from test_gpu_stream import check_fp8

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129, 2, 260]
FORMS = range(4)


@pytest.fixture(autouse=True)
def _default_afterwards():
    import paper_2504_14960_amd as moe
    yield
    moe.set_option("gemm_stream", -1)


# less than a step, a step and a part, a block, less than a ring, ten blocks and 48 bytes; columns of less than a block of 16 on
@pytest.fixture(scope="module", params=[(8, 16), (56, 264), (64, 64), (136, 1416), (664, 72)], ids=str)
def case(request):
    H, F = request.param
    return bf16_case(H=H, F=F, E=len(EDGES), counts=EDGES, seed=7500 + H)


@pytest.mark.parametrize("form", FORMS)
def test_every_form_against_the_oracle(case, form):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = case
    moe.set_option("gemm_stream", 20 + form)
    h, y = bf16_run(x_perm, offsets, inp, 0)
    assert_close(h, h_ref, True, "h")
    assert_close(y, y_ref, True, "y_perm")


@pytest.mark.parametrize("form", FORMS)
def test_every_form_with_the_rounds_of_its_ring(form):
    """Contractions of 40 and 41 blocks: each ring more than twice round, a stage of two blocks left half empty."""
    import paper_2504_14960_amd as moe
    for H, F in ((2560, 128), (128, 2624)):
        inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=3, counts=[70, 200, 5], seed=7600)
        moe.set_option("gemm_stream", 20 + form)
        h, y = bf16_run(x_perm, offsets, inp, 0)
        assert_close(h, h_ref, True, "h")
        assert_close(y, y_ref, True, "y_perm")


# sizes the large tiles do not take have a fifth form, two workgroups to a compute unit: a part of a block, one, a block and a part,
# its ring of two often round with 16 bytes over; columns that end in each of a wave's blocks
@pytest.mark.parametrize("H,F", [(8, 200), (72, 64), (64, 136), (1416, 1000), (264, 2632)])
def test_form_of_the_odd_sizes(H, F):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=len(EDGES), counts=EDGES, seed=7650 + H)
    moe.set_option("gemm_stream", 24)
    h, y = bf16_run(x_perm, offsets, inp, 0)
    assert_close(h, h_ref, True, "h")
    assert_close(y, y_ref, True, "y_perm")


@pytest.mark.parametrize("form", FORMS)
def test_saving_form_has_the_bits_of_the_plain_one(form):
    import torch
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, _ = bf16_case(H=256, F=384, E=4, counts=[40, 0, 129, 31], seed=7700)
    R = int(offsets[-1])
    dx, off, wg, wu = to_dev(x_perm), to_dev(offsets), to_dev(inp["w_gate"]), to_dev(inp["w_up"])
    bf = dict(dtype=torch.bfloat16, device="cuda")
    h, h2, gu = torch.empty((R, 384), **bf), torch.empty((R, 384), **bf), torch.empty((R, 768), **bf)
    moe.set_option("gemm_stream", 20 + form)
    moe.expert_gate_up(dx, off, wg, wu, h)
    moe.expert_gate_up_saving(dx, off, wg, wu, h2, gu)
    assert torch.equal(h, h2)
    assert_close(to_host(h), h_ref, True, "h")
    x = values(x_perm)
    for e in range(4):
        rows = slice(int(offsets[e]), int(offsets[e + 1]))
        want = np.concatenate([x[rows] @ values(inp[w])[e].T for w in ("w_gate", "w_up")], axis=1)
        got = values(to_host(gu))[rows]
        # one rounding to bf16, 2^-9 at most
        assert np.abs(got - want).max(initial=0.0) <= 2.0 ** -8 * np.abs(want).max(initial=0.0)


@pytest.fixture(scope="module", params=[(256, 1408), (1536, 256), (256, 5248)], ids=str)
def fp8(request):
    H, F = request.param
    return fp8_case(seed=7800 + H, H=H, F=F, E=len(EDGES), counts=EDGES)


@pytest.mark.parametrize("form", FORMS)
def test_every_form_in_fp8(fp8, form):
    check_fp8(fp8, 20 + form)


# the last stage of the 128 x 128 form in each slot of its ring (H = 640: the first, which the scratch of amax shares; 768: the loads past
# the last stage end there); tiles of up to 64 rows, whose upper waves have nothing to multiply, and fuller ones
@pytest.mark.parametrize("H", [512, 640, 768, 896])
def test_amax_of_every_last_stage(H):
    c = fp8_case(seed=7900 + H, H=H, F=2816, E=8, counts=[64, 20, 100, 33, 64, 1, 128, 190])
    for form in FORMS:
        for _ in range(3):
            check_fp8(c, 20 + form)


# the forms chosen by size on both sides of one round of workgroups (256 compute units), in odd sizes and FP8
@pytest.mark.parametrize("F", [1000, 1992, 3192, 3400, 6504])
def test_chosen_form_around_one_round(F):
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=264, F=F, E=8, counts=[64, 20, 100, 33, 64, 1, 128, 90], seed=8000 + F)
    h, y = bf16_run(x_perm, offsets, inp, 0)
    assert_close(h, h_ref, True, "h")
    assert_close(y, y_ref, True, "y_perm")


@pytest.mark.parametrize("F", [1408, 2816, 3328, 6656])
def test_chosen_form_around_one_round_in_fp8(F):
    check_fp8(fp8_case(seed=8100 + F, H=512, F=F, E=8, counts=[64, 20, 100, 33, 64, 1, 128, 90]), -1)
