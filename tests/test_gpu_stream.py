"""The weight-streaming expert kernel at the sizes where it can go wrong: the row counts at which a tile changes its
form (16, 32, 64, 128), contractions that end inside a 128-byte block or hold none at all, output columns that end
inside a block of 16, and sizes that select every width of workgroup."""
import numpy as np
import pytest

import oracle
from helpers import assert_close, to_dev, to_host, values
from test_gpu_experts import _case as bf16_case, _run as bf16_run
from test_gpu_fp8 import _case as fp8_case, _check_h_codes, _run as fp8_run

pytestmark = pytest.mark.gpu

EDGES = [1, 16, 17, 32, 33, 0, 64, 65, 128, 129, 2, 260]


@pytest.fixture(autouse=True)
def _always_stream():
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 1)
    yield
    moe.set_option("gemm_stream", -1)


@pytest.mark.parametrize("H,F,counts,bf16", [
    (64, 64, EDGES, True),             # one whole block of the contraction
    (8, 16, EDGES, True),              # less than one block, fewer columns than a block of 16 twice over
    (136, 1416, EDGES, True),          # wide first product, narrow second one; remainders on both axes
    (3000, 72, EDGES, True),           # the other way round
    (1000, 200, EDGES, True),
    (1048, 640, [40, 3], True),        # few workgroups: the waves share the contraction
    (2048, 520, [64], True),
    (1536, 512, [1, 0, 3, 12], True),  # at most 16 rows in all
    (72, 16384, [5, 9], True),         # the same, many columns
    (4, 8, EDGES, False),              # fp32: 16 bytes per row
    (100, 260, EDGES, False),
    (1028, 36, [7, 2], False),
])
def test_stream_against_the_oracle(H, F, counts, bf16):
    pad = 0 if sum(counts) <= 16 else 5
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=len(counts), counts=counts, bf16=bf16, seed=6300 + H, r_pad=pad)
    R = int(offsets[-1])
    h, y = bf16_run(x_perm, offsets, inp, 0, r_max=R + pad)
    # fp32: sums of at most 1028 terms, sqrt(1028) * 6e-8 = 2e-6 relative, within the bar's 1e-5
    assert_close(h[:R], h_ref, bf16, "h")
    assert_close(y[:R], y_ref, bf16, "y_perm")
    assert not h[R:].any() and not y[R:].any()     # rows past the last expert stay untouched


@pytest.mark.parametrize("H,F,counts", [(256, 1408, EDGES), (1536, 256, EDGES), (2304, 256, [40, 3]), (512, 768, [1, 0, 3, 12])])
def test_stream_fp8_against_the_oracle(H, F, counts):
    c = fp8_case(seed=6500 + H, H=H, F=F, E=len(counts), counts=counts)
    h, y, amax = fp8_run(c, r_pad=0 if sum(counts) <= 16 else 5)
    R = c["R"]
    _check_h_codes(h[:R], c["ref"].hq, "h codes")
    assert abs(amax - c["ref"].amax_h) <= 1e-5 * c["ref"].amax_h
    assert_close(y[:R], c["ref"].y, True, "y_perm")
    assert not h[R:].any() and not y[R:].any()


# Contractions that go round every ring of stages at least twice: up to eight stages of KS = 8 / FB blocks of 128 bytes (one
# from 64 weight rows on), and 2 x 4 blocks per wave in the form without a ring.  69 blocks and 48 bytes in bf16.
LONG = [5, 16, 17, 30, 33, 0, 64, 65, 128, 129]


@pytest.fixture(scope="module", params=["gate_up", "down"])
def long_contraction(request):
    H, F = (4440, 200) if request.param == "gate_up" else (200, 4440)
    return {len(c): bf16_case(H=H, F=F, E=len(c), counts=c, seed=6700 + H) for c in (LONG, [1, 0, 3, 12])}


@pytest.mark.parametrize("blocks", [1, 2, 4, 8])
@pytest.mark.parametrize("experts", [len(LONG), 4])      # 4: at most 16 rows in all
def test_every_width_goes_round_its_ring(long_contraction, experts, blocks):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = long_contraction[experts]
    moe.set_option("gemm_stream", 10 + blocks)
    h, y = bf16_run(x_perm, offsets, inp, 0)
    assert_close(h, h_ref, True, "h")
    assert_close(y, y_ref, True, "y_perm")


def check_fp8(c, option):
    """The kernel form `option` on an FP8 case of many sums: y against the oracle, h against the large tiles' h.

    The matrix instruction's own sums of E4M3 products are some 1e-5 off in every kernel: more than a step of the codes for one
    small h in a million.  Between two kernels the order of at most 66 additions remains, sqrt(66) * 6e-8 = 5e-7 relative in
    each of g and u."""
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 0)
    h_large, _, amax_large = fp8_run(c)
    moe.set_option("gemm_stream", option)
    h, y, amax = fp8_run(c)
    _check_h_codes(h, h_large, "h codes")
    assert abs(amax - amax_large) <= 1e-6 * amax_large
    assert_close(y, c["ref"].y, True, "y_perm")


@pytest.fixture(scope="module", params=["gate_up", "down"])
def long_contraction_fp8(request):
    H, F = (8448, 256) if request.param == "gate_up" else (256, 8448)      # 66 blocks
    return {len(c): fp8_case(seed=6800 + H, H=H, F=F, E=len(c), counts=c) for c in (LONG, [1, 0, 3, 12])}


@pytest.mark.parametrize("blocks", [1, 2, 4, 8])
@pytest.mark.parametrize("experts", [len(LONG), 4])
def test_every_width_goes_round_its_ring_in_fp8(long_contraction_fp8, experts, blocks):
    check_fp8(long_contraction_fp8[experts], 10 + blocks)


@pytest.mark.parametrize("blocks", [1, 2, 4, 8])
@pytest.mark.parametrize("H,F", [(1100, 68), (68, 1100)])      # 34 blocks and 48 bytes
def test_every_width_goes_round_its_ring_in_fp32(H, F, blocks):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=len(LONG), counts=LONG, bf16=False, seed=6900 + H)
    moe.set_option("gemm_stream", 10 + blocks)
    h, y = bf16_run(x_perm, offsets, inp, 0)
    # sums of 1100 terms: sqrt(1100) * 6e-8 = 2e-6 relative, within the bar's 1e-5
    assert_close(h, h_ref, False, "h")
    assert_close(y, y_ref, False, "y_perm")


def test_saving_form_and_both_kernels_agree():
    """The pre-activations are those behind h, and the large-tile kernel's results differ by rounding only."""
    import torch
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, _ = bf16_case(H=256, F=384, E=len(EDGES), counts=EDGES, seed=6600)
    R = int(offsets[-1])
    x, off = to_dev(x_perm), to_dev(offsets)
    wg, wu, wd = (to_dev(inp[k]) for k in ("w_gate", "w_up", "w_down"))
    out = {}
    for stream in (1, 0):
        moe.set_option("gemm_stream", stream)
        gu = torch.zeros((R, 768), dtype=torch.bfloat16, device="cuda")
        h, h2 = (torch.zeros((R, 384), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        moe.expert_gate_up_saving(x, off, wg, wu, h, gu)
        moe.expert_gate_up(x, off, wg, wu, h2)
        torch.cuda.synchronize()
        assert torch.equal(h, h2)
        assert_close(to_host(h), h_ref, True, f"h (stream {stream})")
        out[stream] = values(to_host(gu))
    # one rounding each: at most a unit in the last place (2^-8 relative) where the sums straddle a boundary
    assert np.abs(out[0] - out[1]).max() <= np.abs(out[0]).max() * 2.0 ** -7
    assert np.linalg.norm(out[0] - out[1]) <= 1e-3 * np.linalg.norm(out[0])


@pytest.mark.parametrize("H,F,rows", [(8, 16, 30000), (72, 64, 60), (64, 72, 9), (64, 64, 30000)])
def test_silu_is_the_plain_kernels(H, F, rows):
    """silu over the bf16 numbers of [-100, 100], with g and u formed without rounding: the bits of the plain FMA kernel,
    for the shapes that the persistent large tiles do not take (many rows, some sixty, at most sixteen; H = 64)."""
    import torch
    import paper_2504_14960_amd as moe
    g = np.arange(0x10000, dtype=np.uint32).astype(np.uint16)
    g = g[(g & 0x7FFF) <= 0x42C8]                      # |g| <= 100
    g = g[np.linspace(0, g.size - 1, rows).astype(int)]
    x = np.zeros((rows, H), np.uint16)
    x[:, 0], x[:, 1] = g, 0x3F80                       # g and 1
    w = np.zeros((2, F, H), np.uint16)
    w[0, :, 0] = w[1, :, 1] = 0x3F80
    out = []
    for variant in (0, 99):
        h = torch.zeros((rows, F), dtype=torch.bfloat16, device="cuda")
        moe.set_option("gemm_variant", variant)
        try:
            moe.expert_gate_up(to_dev(x), to_dev(np.array([0, rows], np.int32)), to_dev(w[:1]), to_dev(w[1:]), h)
            torch.cuda.synchronize()
        finally:
            moe.set_option("gemm_variant", 0)
        out.append(to_host(h))
    np.testing.assert_array_equal(out[0], out[1])
