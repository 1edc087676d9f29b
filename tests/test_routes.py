"""Which kernels a layer runs on, told by the workspace, for layers that several could take."""
import pytest

from paper_2209_03704_amd import binding as kst
from test_split_plans import split_forward_bytes


@pytest.mark.parametrize("shape", [(3, 854, 480, 8, 5, 1), (2, 1022, 510, 9, 5, 2)])
def test_large_layers_of_few_positions_and_ragged_channels_stay_on_the_split_kernels(shape):
    """... whose positions the position-block kernel could take too: 76 against 134 us on the first."""
    assert kst.kst_workspace_bytes_padded(*shape, kst.KST_F32) == split_forward_bytes(*shape)


@pytest.mark.parametrize("shape,repacked", [
    ((9, 128, 91, 26, 3, 2), True),
    ((33, 64, 3, 32, 4, 2), False),       # three output channels: the tap-major kernel, no scratch
    ((46, 248, 3, 11, 4, 2), True),       # ... many steps of the direct kernel
    ((52, 32, 3, 31, 5, 2), False),       # ... few
])
def test_repacked_fp32_input(shape, repacked):
    B, Cin, Cout, N, n, P = shape
    parts = B * -(-Cin // 16) * 3 * (N + 2 * ((P + 1) // 2)) ** 2 * 32
    assert (kst.kst_workspace_bytes_padded(*shape, kst.KST_F32) >= parts) == repacked
