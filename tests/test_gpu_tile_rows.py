"""The heights of the large expert tiles (256, 192 or 128 rows, chosen on the device): row counts on both sides of each, and
the same bits from all of them."""
import numpy as np
import pytest

import oracle
import test_gpu_backward as backward
from helpers import assert_close, values
from test_gpu_experts import _case as bf16_case, _run as bf16_run
from test_gpu_fp8 import _case as fp8_case, _run as fp8_run

pytestmark = pytest.mark.gpu

# rows of the experts: edges of the three heights, of two tiles of each, an expert without rows
EDGES = [1, 127, 128, 129, 0, 191, 192, 193, 255, 256, 257, 383, 385, 511, 513]


@pytest.fixture(autouse=True)
def _large_tiles():
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 0)
    yield
    moe.set_option("gemm_stream", -1)
    moe.set_option("gemm_tile_rows", 0)


def _each_height(run):
    import paper_2504_14960_amd as moe
    out = []
    for rows in (256, 192, 128, 0):
        moe.set_option("gemm_tile_rows", rows)
        out.append(run())
    return out


# one N-tile and several, the least contraction (two k-tiles) and a ragged number of columns; 32 experts: contiguous shares
@pytest.mark.parametrize("H,F,counts", [(128, 128, EDGES), (320, 576, EDGES), (1024, 192, EDGES), (192, 320, EDGES + [40] * 17)])
def test_heights_against_the_oracle_and_each_other(H, F, counts):
    inp, x_perm, offsets, h_ref, y_ref = bf16_case(H=H, F=F, E=len(counts), counts=counts, bf16=True, seed=8100 + H, r_pad=5)
    R = int(offsets[-1])
    got = _each_height(lambda: bf16_run(x_perm, offsets, inp, 0, r_max=R + 5))
    for h, y in got:
        assert not h[R:].any() and not y[R:].any()     # rows past the last expert stay untouched
        np.testing.assert_array_equal(h, got[0][0])
        np.testing.assert_array_equal(y, got[0][1])
    assert_close(got[0][0][:R], h_ref, True, "h")
    assert_close(got[0][1][:R], y_ref, True, "y_perm")


@pytest.mark.parametrize("H,F,counts", [(256, 256, EDGES), (384, 640, EDGES), (256, 384, EDGES + [40] * 17)])
def test_fp8_heights_against_the_oracle_and_each_other(H, F, counts):
    c = fp8_case(seed=8200 + H, H=H, F=F, E=len(counts), counts=counts)
    R = c["R"]
    got = _each_height(lambda: fp8_run(c, r_pad=5))
    for h, y, amax in got:
        assert not h[R:].any() and not y[R:].any()
        np.testing.assert_array_equal(h, got[0][0])
        np.testing.assert_array_equal(y, got[0][1])
        assert amax == got[0][2]
    # codes as in test_gpu_fp8, and near zero the absolute error of the matrix instruction's sums of E4M3 products as well:
    # 1.2e-5 of the largest h (its measured error in max |h|), whose code is at most 448
    code, want = oracle.fp8_decode(got[0][0][:R]), oracle.fp8_decode(c["ref"].hq)
    assert (got[0][0][:R] != c["ref"].hq).mean() <= 3e-3
    assert (np.abs(code - want) <= np.maximum(np.abs(want) * 2.0 ** -3, 2.0 ** -9) + 448 * 1.2e-5).all()
    # the 2-norm bar of assert_close; its bar for the largest difference is for outputs whose inputs are the same: an h code on
    # the neighbouring step moves a whole row of y, and with 4000 rows one of them has several such codes
    y = values(got[0][1][:R])
    assert np.linalg.norm(y - c["ref"].y) <= 5e-3 * np.linalg.norm(c["ref"].y)


# few rows per expert, and on average more than 640
MANY = [700, 1, 1300, 257, 0, 2000]


@pytest.fixture(scope="module", params=[EDGES, MANY], ids=["few", "many"])
def two_regimes(request):
    return bf16_case(H=192, F=320, E=len(request.param), counts=request.param, bf16=True, seed=8300, r_pad=5)


@pytest.mark.parametrize("workgroups", [8, 13, 0])
def test_heights_several_tiles_per_workgroup(two_regimes, workgroups):
    """A workgroup walks from tile to tile at every height, with the bits of one tile per workgroup."""
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = two_regimes
    R = int(offsets[-1])
    want_h, want_y = bf16_run(x_perm, offsets, inp, 0, r_max=R + 5)
    assert_close(want_h[:R], h_ref, True, "h")
    assert_close(want_y[:R], y_ref, True, "y_perm")
    moe.set_option("gemm_workgroups", workgroups)
    try:
        for h, y in _each_height(lambda: bf16_run(x_perm, offsets, inp, 0, r_max=R + 5)):
            np.testing.assert_array_equal(h, want_h)
            np.testing.assert_array_equal(y, want_y)
    finally:
        moe.set_option("gemm_workgroups", 0)


@pytest.mark.parametrize("workgroups", [8, 13])
def test_fp8_heights_several_tiles_per_workgroup(workgroups):
    import paper_2504_14960_amd as moe
    c = fp8_case(seed=8400, H=256, F=384, E=len(EDGES), counts=EDGES)
    want = fp8_run(c, r_pad=5)
    moe.set_option("gemm_workgroups", workgroups)
    try:
        for got in _each_height(lambda: fp8_run(c, r_pad=5)):
            np.testing.assert_array_equal(got[0], want[0])
            np.testing.assert_array_equal(got[1], want[1])
            assert got[2] == want[2]
    finally:
        moe.set_option("gemm_workgroups", 0)


# the saving forward, dh with the SwiGLU's derivative and dx, at the heights that the sizes would not choose
@pytest.mark.parametrize("rows", [256, 192, 128])
@pytest.mark.parametrize("saved", [False, True])
def test_backward(rows, saved):
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_tile_rows", rows)
    backward.test_expert_ffn_backward_against_oracle(256, 384, 7, [1, 130, 0, 192, 193, 257, 386], saved, 0)


@pytest.mark.parametrize("rows,workgroups", [(256, 8), (192, 8), (192, 0), (128, 8), (128, 0)])
@pytest.mark.parametrize("saved", [False, True])
def test_backward_of_many_rows(rows, workgroups, saved):
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_tile_rows", rows)
    moe.set_option("gemm_workgroups", workgroups)
    try:
        backward.test_expert_ffn_backward_against_oracle(256, 384, len(MANY), MANY, saved, 0)
    finally:
        moe.set_option("gemm_workgroups", 0)


def test_tile_rows_option_refuses_other_values():
    import paper_2504_14960_amd as moe
    for bad in (-1, 1, 64, 160, 512):
        with pytest.raises(Exception, match="gemm_tile_rows"):
            moe.set_option("gemm_tile_rows", bad)
