"""The perceptron's workspace: no larger than what the layers need one by one, but for the operands' rounding to
whole tiles of rows and the packed weights."""
import ctypes

import pytest

from paper_1403_7394_amd import hap
from test_gpu_mlp_fused import layered_bytes


@pytest.mark.parametrize("n_in,hidden,n_out,rows", [(32, 128, 3, 65536), (32, 256, 4, 4096), (32, 64, 1, 4000),
                                                    (16, 112, 3, 100000)])
def test_workspace_is_no_larger_than_the_layers_need(n_in, hidden, n_out, rows):
    b = ctypes.c_size_t()
    assert hap.load().hap_mlp_workspace_size(n_in, hidden, n_out, rows, ctypes.byref(b)) == 0
    whole = (rows + 31) // 32 * 32
    # four operands of hidden units in FP32, the inputs padded to 32, the outputs to 16, a sum per tile
    bound = whole * (4 * hidden * 4 + 32 * 4 + 16 * 4) + whole // 32 * 8 + 8 * 256
    assert b.value <= max(layered_bytes(n_in, hidden, n_out, rows), bound) + 4 * 256 * (256 + 32)
