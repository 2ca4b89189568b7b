"""The small shapes of the expert tests on the large-tile kernels too: by size they go to the streaming kernels."""
import pytest

import test_gpu_backward as backward
import test_gpu_experts as experts
import test_gpu_fp8 as fp8
from test_gpu_experts import ragged_case    # noqa: F401 (fixtures)
from test_gpu_fp8 import ragged_fp8         # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _large_tiles():
    import paper_2504_14960_amd as moe
    moe.set_option("gemm_stream", 0)
    yield
    moe.set_option("gemm_stream", -1)


def test_ragged_experts(ragged_case):
    experts.test_every_kernel_variant_on_ragged_experts(ragged_case, 0)


def test_deep_contraction_and_fine_grained_experts():
    experts.test_deep_contraction_and_fine_grained_experts(0)


def test_experts_with_more_m_tiles_than_one_scheduler_group():
    experts.test_experts_with_more_m_tiles_than_one_scheduler_group(0)


def test_rows_past_the_last_expert():
    experts.test_rows_past_the_last_expert_are_untouched_and_result_is_reproducible()


def test_all_experts_empty():
    experts.test_all_experts_empty_is_a_no_op()


def test_clock_sample(ragged_case):
    experts.test_clock_sample_reports_a_plausible_shader_clock_and_leaves_the_results_alone(ragged_case)


def test_fp8_ragged_experts(ragged_fp8):
    fp8.test_ffn_fp8_on_ragged_experts(ragged_fp8)


def test_fp8_down(ragged_fp8):
    fp8.test_down_fp8_on_the_oracles_h_codes(ragged_fp8)


def test_fp8_deep_contraction_and_many_small_experts():
    fp8.test_ffn_fp8_deep_contraction_and_many_small_experts()


def test_fp8_reproducible_and_empty():
    fp8.test_ffn_fp8_is_reproducible_and_handles_empty_input()


# the forward that keeps its pre-activations, the plain products of the backward, dh with and without the SwiGLU's derivative
@pytest.mark.parametrize("H,F,E,counts", [(256, 384, 6, [700, 0, 1, 300, 513, 86]), (128, 128, 3, [64, 130, 5]),
                                          (384, 256, 64, None), (640, 384, 2, [1300, 77])])
@pytest.mark.parametrize("saved", [False, True])
def test_backward(H, F, E, counts, saved):
    backward.test_expert_ffn_backward_against_oracle(H, F, E, counts, saved, 0)


@pytest.mark.parametrize("base,kw", [("mixtral8x22b", dict(T=640, H=256, F=384)), ("tokendrop", dict(T=1536, H=256, F=256))])
def test_training_step(base, kw):
    backward.test_layer_training_step_in_two_calls(base, kw)
