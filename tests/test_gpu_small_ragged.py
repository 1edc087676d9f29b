"""fp32 layers of few positions whose channel counts are no whole groups of four, on position blocks of 16: against the
oracle, and bit for bit on integers with guard words around the output."""
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import TOL, check_exact_with_guards, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SHAPES = [
    (1, 153, 40, 16, 3, 2),     # one input channel in the last chunk, whole output groups
    (1, 270, 175, 8, 4, 2),     # four waves per workgroup, last group moved back by one channel
    (1, 87, 66, 4, 5, 1),       # 66 = 64 + 2: the second block's group begins in the first one's channels
    (1, 94, 65, 4, 5, 0),       # ... by three channels
    (3, 50, 67, 5, 4, 3),       # several items, odd padding factor
    (2, 17, 19, 9, 3, 1),
    (2, 40, 18, 20, 3, 2),      # fewer than 64 input channels
    (1, 128, 6, 12, 4, 2),      # few output channels
    (1, 201, 5, 8, 5, 2),
    (1, 163, 4, 9, 3, 0),
    (1, 143, 3, 7, 5, 1),       # ... fewer than a group
    (1, 1001, 2, 5, 4, 2),
]


@pytest.mark.parametrize("B,Cin,Cout,N,n,P", SHAPES)
def test_ragged_channels_on_position_blocks(B, Cin, Cout, N, n, P):
    need = kst.kst_workspace_bytes_padded(B, Cin, Cout, N, n, P, kst.KST_F32)
    M = kst.kst_out_size_padded(N, n, P)
    assert need > 0 and need % (B * Cout * M * M * 4) == 0             # partial outputs of a split reduction
    layer = wl.Layer("small_ragged", B, Cin, Cout, N, n, "f32", "relu_normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 3100 + Cin)
    seg = kst.kst_segregate_weights(w.to(DEV))
    got = kst.kst_forward_seg_padded(x.to(DEV), seg, Cout, n, P)
    e = rel_err(got.cpu().numpy(), oracle.forward(wl.to_f64(x), wl.to_f64(w), P))
    assert e <= TOL["f32"], "rel err %.3e" % e
    check_exact_with_guards(wl.Layer("small_ragged_int", B, Cin, Cout, N, n, "f32", "integer"), kst.KST_PATH_AUTO, 3200 + Cin, P=P)
    # Values that are not finite stay where they belong: the last input channel shares its chunk with channels that are not.
    x[0, Cin - 1, 1, 1] = float("inf")
    w[Cout - 1, 0, 0, 0] = float("nan")
    seg = kst.kst_segregate_weights(w.to(DEV))
    got = kst.kst_forward_seg_padded(x.to(DEV), seg, Cout, n, P)
    plain = kst.kst_forward_seg_padded(x.to(DEV), seg, Cout, n, P, path=kst.KST_PATH_DIRECT)
    assert torch.equal(torch.isfinite(got[:, :Cout - 1]), torch.isfinite(plain[:, :Cout - 1]))


def test_less_scratch_than_the_partial_outputs():
    """The kernels that ran these layers before, where their scratch is enough."""
    B, Cin, Cout, N, n, P = 1, 143, 3, 7, 5, 1
    x = torch.randn(B, Cin, N, N, device=DEV)
    seg = kst.kst_segregate_weights(torch.randn(Cout, Cin, n, n, device=DEV))
    need = kst.kst_workspace_bytes_padded(B, Cin, Cout, N, n, P, kst.KST_F32)
    short = kst.kst_forward_seg_padded(x, seg, Cout, n, P, ws=torch.empty(need - 1, dtype=torch.uint8, device=DEV))
    assert torch.equal(short, kst.kst_forward_seg_padded(x, seg, Cout, n, P, path=kst.KST_PATH_DIRECT))
