"""One input channel, weights as they come: the same bits as from segregated weights."""
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import TOL, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("B,Cout,N,n", [(1, 1, 32, 3), (2, 3, 17, 4), (3, 2, 24, 5), (1, 5, 9, 7), (2, 1, 12, 1), (1, 2, 13, 2), (4, 1, 31, 6),
                                        (1, 1, 6, 9), (2, 2, 100, 3)])
def test_whole_call_of_one_channel(B, Cout, N, n, dtype):
    layer = wl.Layer("plain_weights", B, 1, Cout, N, n, dtype, "normal", w_std=0.2)
    x, w = wl.make_tensors(layer, 3100 + N)
    got = kst.kst_forward(x.to(DEV), w.to(DEV))
    seg = kst.kst_forward_seg(x.to(DEV), kst.kst_segregate_weights(w.to(DEV)), Cout, n)
    assert torch.equal(got, seg)
    assert rel_err(got.cpu().numpy(), oracle.forward(wl.to_f64(x), wl.to_f64(w), 0)) <= TOL[dtype]
