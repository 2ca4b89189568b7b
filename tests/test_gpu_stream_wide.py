"""The wide form of the weight-streaming expert kernel: row counts on both sides of its tile forms, partial blocks of the
contraction, every number of weight rows per workgroup, and the contraction in every number of parts."""
import numpy as np
import pytest

from moe_inputs import get_config, make_layer_inputs
from helpers import assert_close, guard_margins, to_dev, to_host, values
from test_gpu_experts import _case as bf16_case, _run as bf16_run
from test_gpu_fp8 import _case as fp8_case, _check_h_codes, _run as fp8_run
from test_gpu_layer import oracle_layer
from test_gpu_stream import EDGES, check_fp8

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _always_wide():
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 2)
    yield
    moe.set_option("gemm_stream", -1)


@pytest.mark.parametrize("H,F,counts", [
    (64, 64, EDGES),               # one whole block of the contraction; fewer columns than a workgroup's
    (8, 16, EDGES),                # no whole block at all
    (136, 1416, EDGES),            # remainders on both axes
    (3000, 72, EDGES),             # the other way round
    (1088, 640, [40, 3]),          # a contraction that is not a multiple of the ring's stages
    (256, 20480, [65]),            # one round of workgroups of 160 weight rows
    (14336, 256, [5, 90, 7]),
])
def test_wide_against_the_oracle(H, F, counts):
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=len(counts), counts=counts, bf16=True, seed=7300 + H, r_pad=5)
    R = int(offsets[-1])
    h, y = bf16_run(x_perm, offsets, inp, 0, r_max=R + 5)
    assert_close(h[:R], h_ref, True, "h")
    assert_close(y[:R], y_ref, True, "y_perm")
    assert not h[R:].any() and not y[R:].any()     # rows past the last expert stay untouched


@pytest.mark.parametrize("H,F,counts", [(256, 1408, EDGES), (1536, 256, EDGES), (512, 768, [1, 0, 3, 12])])
def test_wide_fp8_against_the_oracle(H, F, counts):
    c = fp8_case(seed=7500 + H, H=H, F=F, E=len(counts), counts=counts)
    h, y, amax = fp8_run(c, r_pad=5)
    R = c["R"]
    _check_h_codes(h[:R], c["ref"].hq, "h codes")
    assert abs(amax - c["ref"].amax_h) <= 1e-5 * c["ref"].amax_h
    assert_close(y[:R], c["ref"].y, True, "y_perm")
    assert not h[R:].any() and not y[R:].any()


UNITS = [3, 4, 5, 6, 7, 8]      # blocks of 32 weight rows per workgroup; the last has no idle wave


@pytest.fixture(scope="module", params=[(2184, 1416), (1416, 2184)])
def ragged(request):
    """34 blocks of 128 bytes and 16 bytes, 22 and 16: each ring of eight stages is gone round twice; the columns end inside a
    workgroup's and inside a block of 16."""
    H, F = request.param
    return bf16_case(H=H, F=F, E=len(EDGES), counts=EDGES, seed=7600 + H, r_pad=5)


@pytest.mark.parametrize("units", UNITS)
def test_every_number_of_weight_rows(ragged, units):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = ragged
    R = int(offsets[-1])
    moe.set_option("gemm_stream", 100 + units)
    h, y = bf16_run(x_perm, offsets, inp, 0, r_max=R + 5)
    assert_close(h[:R], h_ref, True, "h")
    assert_close(y[:R], y_ref, True, "y_perm")
    assert not h[R:].any() and not y[R:].any()


@pytest.mark.parametrize("units", UNITS)
def test_every_number_of_weight_rows_in_fp8(units):
    check_fp8(fp8_case(seed=7650, H=2304, F=640, E=len(EDGES), counts=EDGES), 100 + units)


def _layer_case(T, H, F, Fs, E, K):
    cfg = get_config("qwen2_57b_a14b").scaled(T=T, H=H, F=F, E=E, K=K, shared_F=Fs, seed=7700 + T)
    inp = make_layer_inputs(cfg)
    guard_margins(inp, K)
    return inp, oracle_layer(inp, 0)


def _check_split_layer(case, parts):
    """With the workspace that is asked for, `parts` bytes beyond the intermediates, and with one too small for the partial
    sums: both are the oracle's layer."""
    import torch
    import paper_2504_14960_amd as moe
    inp, want = case
    c = inp.cfg
    d = {k: to_dev(v) for k, v in inp.tensors.items()}
    bias = None if inp.bias is None else to_dev(inp.bias)
    nbytes = moe.layer_workspace_bytes(c.T, c.H, c.E, c.K, c.F, c.shared_F, 0, moe.MOE_BF16)
    lay = moe.layer_workspace_layout(c.T, c.H, c.E, c.K, c.F, c.shared_F, 0, moe.MOE_BF16)
    end = (lay["shared_y"] + c.T * c.H * 2 + 255) // 256 * 256
    assert nbytes - end == parts, "the shape is meant to want these partial sums"
    out = []
    for size in (nbytes, end):
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")      # NaN patterns: nothing unwritten is added
        y = torch.empty_like(d["x"])
        moe.layer_forward(d["x"], d["w_router"], bias, d["w_gate"], d["w_up"], d["w_down"], d["ws_gate"], d["ws_up"],
                          d["ws_down"], c.K, c.renormalize, 0, y, ws)
        torch.cuda.synchronize()
        out.append(values(to_host(y)))
        assert_close(to_host(y), want.y, True, f"y ({size} bytes)")
    # the same products with their sums in another order: half a unit in the last place of bf16 here and there
    assert np.linalg.norm(out[0] - out[1]) <= 2e-3 * np.linalg.norm(out[0])


@pytest.mark.parametrize("T,H,F,Fs,E,K,parts", [
    (40, 512, 128, 4096, 4, 2, 4 * 40 * 512 * 4),          # the down projection in four parts
    (150, 2560, 64, 1024, 6, 2, 2 * 150 * 1024 * 8),       # gate/up in two; two M-tiles
])
def test_split_contraction_in_the_layer(T, H, F, Fs, E, K, parts):
    _check_split_layer(_layer_case(T, H, F, Fs, E, K), parts)


# 260 blocks of 128 bytes and 16 bytes: no whole number of blocks to a part, and the partial block goes to the last one; the
# other axis ends inside a workgroup's columns
@pytest.fixture(scope="module", params=[(40, 16648, 328), (40, 328, 16648), (100, 16648, 328), (130, 328, 16648)])
def long_shared(request):
    T, H, Fs = request.param
    return _layer_case(T, H, 64, Fs, 4, 2)


@pytest.mark.parametrize("units,splits", [(3, 16), (4, 8), (5, 4), (6, 2), (7, 16), (8, 16), (8, 1)])
def test_every_number_of_parts(long_shared, units, splits):
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 100 * splits + units)
    c = long_shared[0].cfg
    per = c.shared_F * 8 if c.H > c.shared_F else c.H * 4         # gate/up with its two sums, or down; the other stays whole
    _check_split_layer(long_shared, splits * c.T * per if splits > 1 else 0)


# the large tiles, contraction in parts: 41 k-tiles, no whole number to a part; rows at the edges of the three tile heights;
# columns that end inside a tile; gate/up (H > Fs) and down
@pytest.fixture(scope="module", params=[(129, 2624, 320), (193, 320, 2624), (257, 2624, 448), (385, 448, 2624)])
def deep_shared(request):
    T, H, Fs = request.param
    return _layer_case(T, H, 64, Fs, 4, 2)


@pytest.mark.parametrize("splits,rows", [(2, 0), (3, 256), (3, 192), (3, 128), (5, 0)])
def test_large_tiles_in_parts(deep_shared, splits, rows):
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 2000 + splits)
    moe.set_option("gemm_tile_rows", rows)
    try:
        c = deep_shared[0].cfg
        _check_split_layer(deep_shared, splits * c.T * (c.shared_F * 8 if c.H > c.shared_F else c.H * 4))
    finally:
        moe.set_option("gemm_tile_rows", 0)


# from tile to tile the number of k-tiles (2624 elements in 3 parts: 13 or 14, in 5: 8 or 9) and the plane change
@pytest.mark.parametrize("workgroups", [8, 13])
@pytest.mark.parametrize("splits,rows", [(3, 0), (5, 256), (5, 192), (5, 128)])
def test_large_tiles_in_parts_several_tiles_per_workgroup(deep_shared, splits, rows, workgroups):
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_workgroups", workgroups)
    try:
        test_large_tiles_in_parts(deep_shared, splits, rows)
    finally:
        moe.set_option("gemm_workgroups", 0)
