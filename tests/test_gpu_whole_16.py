"""Whole calls of 16-bit layers whose input is repacked: weights segregated by the same launch, bit for bit what
segregating them first and the segregated entry point give."""
import pytest
import torch

from paper_2209_03704_amd import binding as kst

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Channels that are no whole groups of 8 or 16, a last workgroup of few elements on either side, odd and even padding
# factors, all kernel edges, split reductions, one item and many.
LAYERS = [(24, 100, 52, 19, 3, 1), (1, 600, 33, 9, 4, 0), (5, 17, 130, 16, 5, 2), (3, 200, 3, 30, 4, 3), (40, 64, 64, 7, 3, 0),
          (2, 1000, 257, 6, 5, 2), (130, 20, 16, 12, 4, 1)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("layer", LAYERS)
def test_whole_call_is_the_segregated_one(layer, dtype):
    B, Cin, Cout, N, n, P = layer
    gen = torch.Generator().manual_seed(3 + B)
    for _ in range(2):                                # (the pool's scratch holds the last call's weights)
        x = torch.randn((B, Cin, N, N), generator=gen).to(dtype).to(DEV)
        w = (torch.randn((Cout, Cin, n, n), generator=gen) * 0.05).to(dtype).to(DEV)
        out = kst.kst_forward_padded(x, w, P) if P else kst.kst_forward(x, w)
        assert torch.equal(out, kst.kst_forward_seg_padded(x, kst.kst_segregate_weights(w), Cout, n, P))
