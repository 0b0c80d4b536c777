"""The gradient tests once more from the least workspace, where fp32-arithmetic kernels form their own scores: every feature map,
rotation, split queries with a gradient of their own, cache buffers, ragged and random shapes, inputs that are not finite."""
import pytest

import paper_2604_10103_amd as hf
from test_gpu_backward import (  # noqa: F401
    test_backward_ragged_and_degenerate_sizes, test_backward_seeded_random_shapes,
    test_bf16_kernel_choices_and_key_blocks_that_are_no_multiple_of_a_tile, test_gradients_in_a_cache_buffer_layout,
    test_gradients_of_the_whole_path_match_oracle, test_split_queries_no_state_and_dense_window)
from test_gpu_nonfinite import test_gradients_of_other_blocks  # noqa: F401
from test_gpu_split import test_forward_and_gradients, test_fp32_products_at_either_number_of_rows  # noqa: F401
from test_gpu_wide import test_forward_and_gradients_at_tile_edges  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def least_workspace(monkeypatch):
    asked = []

    def least(*args):
        asked.append(args)
        return hf.hf_bwd_least_workspace_bytes(*args)

    monkeypatch.setattr(hf, "hf_bwd_workspace_bytes", least)
    yield
    assert asked
