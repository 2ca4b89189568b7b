"""fp32 expert products on the bf16 matrix instruction, every form of their tiles: row counts around the edges of the tiles, columns
and contractions that end inside a tile, a block or a group's turn, and operands that three bf16 parts cannot stand for."""
import numpy as np
import pytest

import oracle
from helpers import assert_close, to_dev, to_host
from test_gpu_experts import _case, _run

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 33, 0, 63, 64, 65, 127, 128, 129, 2, 260]


@pytest.fixture(autouse=True)
def _default_afterwards():
    import paper_2504_14960_amd as moe
    yield
    moe.set_option("gemm_stream", -1)


@pytest.fixture(scope="module", params=[(4, 8), (36, 260), (260, 36), (544, 132), (132, 1100)], ids=str)
def case(request):
    H, F = request.param
    return _case(H=H, F=F, E=len(EDGES), counts=EDGES, bf16=False, seed=7100 + H)


@pytest.mark.parametrize("form", range(5))
def test_every_form_against_the_oracle(case, form):
    import paper_2504_14960_amd as moe
    inp, x_perm, offsets, h_ref, y_ref = case
    moe.set_option("gemm_stream", 20 + form)
    R = int(offsets[-1])
    h, y = _run(x_perm, offsets, inp, 0)
    # a sum of 1100 terms is rounded once per 16 of them and its products are 2^-26 off: some 3e-7 relative, within the bar's 1e-5
    assert_close(h[:R], h_ref, False, "h")
    assert_close(y[:R], y_ref, False, "y_perm")


@pytest.mark.parametrize("form", range(5))
def test_infinite_and_nan_rows(form):
    """Infinities, NaN and the largest numbers of a row show in its own results and nowhere else, and are those of fp32."""
    import torch
    import paper_2504_14960_amd as moe
    rng = np.random.default_rng(5)
    R, H, F = 40, 72, 48
    x = rng.standard_normal((R, H)).astype(np.float32)
    x[3, 5] = np.inf
    x[7, 70] = -np.inf
    x[9, 71] = np.nan
    x[11, 0] = 3.4e38          # no bf16 of its own: rounds to infinity
    x[13] *= 1e-36             # the third part is below the normal numbers
    wg, wu = (rng.standard_normal((1, F, H)).astype(np.float32) * 0.02 for _ in range(2))
    off = torch.tensor([0, R], dtype=torch.int32).cuda()
    h = torch.empty((R, F), dtype=torch.float32, device="cuda")
    moe.set_option("gemm_stream", 20 + form)
    moe.expert_gate_up(to_dev(x), off, to_dev(wg), to_dev(wu), h)
    got = to_host(h)
    with np.errstate(all="ignore"):
        g, u = (x.astype(np.float64) @ w[0].T.astype(np.float64) for w in (wg, wu))
        want = ((g / (1.0 + np.exp(-g))) * u).astype(np.float32)
    special = [3, 7, 9, 11]
    plain = np.setdiff1d(np.arange(R), special)
    assert np.isfinite(got[plain]).all()
    ordinary = np.setdiff1d(plain, [13])
    assert np.linalg.norm(got[ordinary] - want[ordinary]) <= 1e-5 * np.linalg.norm(want[ordinary])
    for r in (3, 7, 9):
        assert (np.isnan(got[r]) == np.isnan(want[r])).all()
        assert (np.isposinf(got[r]) == np.isposinf(want[r])).all() and (np.isneginf(got[r]) == np.isneginf(want[r])).all()
    # row 11 by its pre-activations near 1e36: g u overflows where it should
    assert (np.isfinite(got[11]) == np.isfinite(want[11])).all()
    # row 13: g u / 2 of two sums of 1e-36 size is zero in fp32
    assert not got[13].any()
    # and its sums, through the second product
    y = torch.empty((R, H), dtype=torch.float32, device="cuda")
    wd = rng.standard_normal((1, H, F)).astype(np.float32) * 0.02
    hh = rng.standard_normal((R, F)).astype(np.float32)
    hh[13] *= 1e-30
    moe.expert_down(to_dev(hh), off, to_dev(wd), y)
    ref = hh.astype(np.float64) @ wd[0].T.astype(np.float64)
    got = to_host(y)
    assert np.linalg.norm(got[13] - ref[13]) <= 1e-5 * np.linalg.norm(ref[13])


def test_chosen_form_keeps_the_results_of_the_fp32_instruction():
    """The same product with the form chosen, on both sides of the line between the two instructions."""
    import paper_2504_14960_amd as moe
    for counts in ([12, 12, 12, 12], [13, 13, 13, 13], [200, 3, 40, 77]):
        inp, x_perm, offsets, h_ref, y_ref = _case(H=200, F=300, E=4, counts=counts, bf16=False, seed=7300)
        for option in (-1, 1):
            moe.set_option("gemm_stream", option)
            h, y = _run(x_perm, offsets, inp, 0)
            assert_close(h, h_ref, False, "h")
            assert_close(y, y_ref, False, "y_perm")


@pytest.mark.parametrize("form", range(5))
def test_operands_below_what_their_parts_can_hold(form):
    """Rows and weights whose third bf16 part is below the smallest bf16 number (from some 1e-33 down): the results keep the bits of
    fp32, and the rows beside them keep their own."""
    import torch
    import paper_2504_14960_amd as moe
    rng = np.random.default_rng(6)
    R, H, F = 80, 96, 48
    h = rng.standard_normal((2 * R, F)).astype(np.float32)
    wd = rng.standard_normal((2, H, F)).astype(np.float32)
    wd[1] *= np.float32(1e-36)                      # the second expert: tiny weights
    tiny = {3: 1e-32, 8: 1e-33, 20: 1e-34, 33: 1e-35, 64: 1e-36, 79: 3e-37}
    plain, off = h.copy(), to_dev(np.array([0, R, 2 * R], np.int32))
    for r, s in tiny.items():
        h[r] *= np.float32(s)
    moe.set_option("gemm_stream", 20 + form)
    got = []
    for rows in (h, plain):
        y = torch.empty((2 * R, H), dtype=torch.float32, device="cuda")
        moe.expert_down(to_dev(rows), off, to_dev(wd), y)
        got.append(to_host(y))
    ref = np.concatenate([h[e * R:(e + 1) * R].astype(np.float64) @ wd[e].T.astype(np.float64) for e in range(2)])
    for r in list(tiny) + list(range(R, 2 * R)):
        # sums of 48 terms in fp32: sqrt(48) * 6e-8 = 4e-7
        assert np.linalg.norm(got[0][r] - ref[r]) <= 1e-6 * np.linalg.norm(ref[r]), r
    others = [r for r in range(R) if r not in tiny]
    np.testing.assert_array_equal(got[0][others], got[1][others])
