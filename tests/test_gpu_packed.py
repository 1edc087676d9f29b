"""16-bit layers whose input is repacked, channels of a pixel side by side: against the oracle, bit for bit on integers with
guard words around the output, and against the kernels that take the input as it lies in memory."""
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import TOL, check_exact_with_guards, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {"bf16": kst.KST_BF16, "f16": kst.KST_F16}


def packed_bytes(B, Cin, N, P):
    return B * -(-Cin // 16) * (N + 2 * ((P + 1) // 2)) ** 2 * 32


# Every kernel edge with one and two position blocks per wave and both stage sizes; whole and split reductions; ragged
# channels (an odd number of eights, one channel in the last); odd maps and padding factors; one and few output channels.
SHAPES = [
    (24, 100, 52, 19, 3, 1, "f16"),     # odd map and padding factor, seven chunks of which the last holds four channels
    (5, 37, 70, 13, 4, 0, "bf16"),      # unframed, five channels in the last eight
    (3, 64, 40, 9, 5, 3, "f16"),        # several items per tile, odd padding factor
    (2, 456, 24, 6, 4, 2, "bf16"),      # split reduction, summing pass
    (2, 450, 20, 7, 5, 1, "f16"),       # ... with an odd padding factor
    (40, 24, 64, 40, 3, 0, "bf16"),     # two position blocks per wave, large stages
    (33, 40, 100, 31, 4, 2, "f16"),
    (70, 33, 40, 33, 5, 1, "bf16"),
    (200, 17, 130, 6, 3, 2, "f16"),     # two position blocks, small stages, many items per tile
    (64, 48, 128, 16, 4, 2, "bf16"),
    (40, 16, 128, 18, 5, 0, "f16"),
    (1, 17, 16, 100, 3, 0, "bf16"),     # one position block, large stages
    (2, 20, 16, 60, 4, 3, "f16"),
    (2, 24, 16, 50, 5, 2, "bf16"),
    (90, 16, 16, 2, 3, 1, "f16"),       # the smallest map
    (4, 80, 3, 20, 4, 1, "bf16"),       # three output channels of 32 rows
    (2, 70, 1, 21, 5, 2, "f16"),
]


def _run(layer, P, seed, path=kst.KST_PATH_AUTO, bias=None, act=kst.KST_ACT_NONE):
    x, w = wl.make_tensors(layer, seed)
    seg = kst.kst_segregate_weights(w.to(DEV))
    if bias is None:
        got = kst.kst_forward_seg_padded(x.to(DEV), seg, layer.Cout, layer.n, P, path=path)
    else:
        got = kst.kst_forward_seg_epilogue(x.to(DEV), seg, layer.Cout, layer.n, bias=bias.to(DEV), act=act, P=P, path=path)
    torch.cuda.synchronize()
    return x, w, got


@pytest.mark.parametrize("B,Cin,Cout,N,n,P,dtype", SHAPES)
def test_repacked_input(B, Cin, Cout, N, n, P, dtype):
    need = kst.kst_workspace_bytes_padded(B, Cin, Cout, N, n, P, CODE[dtype])
    assert need >= packed_bytes(B, Cin, N, P)                       # the repacked input is in it
    layer = wl.Layer("packed", B, Cin, Cout, N, n, dtype, "relu_normal", w_std=0.1)
    x, w, got = _run(layer, P, 2100 + N + Cin)
    e = rel_err(got.cpu().numpy(), oracle.forward(wl.to_f64(x), wl.to_f64(w), P))
    assert e <= TOL[dtype], "rel err %.3e" % e
    check_exact_with_guards(wl.Layer("packed_int", B, Cin, Cout, N, n, dtype, "integer"), kst.KST_PATH_AUTO, 2200 + N, P=P)


@pytest.mark.parametrize("act", [kst.KST_ACT_NONE, kst.KST_ACT_RELU, kst.KST_ACT_TANH])
@pytest.mark.parametrize("B,Cin,Cout,N,n,P,dtype", [SHAPES[0], SHAPES[3], SHAPES[5], SHAPES[9]])
def test_repacked_input_epilogue(B, Cin, Cout, N, n, P, dtype, act):
    layer = wl.Layer("packed_epi", B, Cin, Cout, N, n, dtype, "relu_normal", w_std=0.1)
    bias = torch.randn(Cout, generator=torch.Generator().manual_seed(7))
    x, w, got = _run(layer, P, 2300 + N, bias=bias, act=act)
    want = oracle.forward_epilogue(wl.to_f64(x), wl.to_f64(w), wl.to_f64(bias), act, P)
    e = rel_err(got.cpu().numpy(), want)
    assert e <= TOL[dtype], "rel err %.3e" % e


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_repacked_input_not_finite(value):
    """An input value that is not finite reaches the outputs its products are in, and only those; so does a weight."""
    B, Cin, Cout, N, n, P = 2, 21, 20, 11, 3, 1
    layer = wl.Layer("packed_inf", B, Cin, Cout, N, n, "bf16", "normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 2400)
    for hit_x in (True, False):
        a, b = x.clone(), w.clone()
        if hit_x:
            a[1, 20, 5, 4] = value
        else:
            b[19, 20, 1, 1] = value
        seg = kst.kst_segregate_weights(b.to(DEV))
        got = kst.kst_forward_seg_padded(a.to(DEV), seg, Cout, n, P)
        old = kst.kst_forward_seg_padded(a.to(DEV), seg, Cout, n, P, path=kst.KST_PATH_IGEMM)
        assert torch.equal(torch.isfinite(got), torch.isfinite(old)) and not torch.isfinite(got).all()
        assert torch.equal(torch.isnan(got), torch.isnan(old))


def test_less_scratch_than_the_repacked_input():
    """A byte less than the repacked input wants: the kernels that do without, bit for bit; the static entry point too."""
    B, Cin, Cout, N, n, P = 40, 24, 64, 40, 3, 0
    layer = wl.Layer("packed_ws", B, Cin, Cout, N, n, "f16", "relu_normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 2500)
    x, seg = x.to(DEV), kst.kst_segregate_weights(w.to(DEV))
    need = kst.kst_workspace_bytes(B, Cin, Cout, N, n, kst.KST_F16)
    assert kst.kst_workspace_bytes(B, Cin, Cout, N, n, kst.KST_F16, kst.KST_PATH_IGEMM) < need
    old = kst.kst_forward_seg(x, seg, Cout, n, path=kst.KST_PATH_IGEMM)
    assert torch.equal(kst.kst_forward_seg(x, seg, Cout, n, ws=torch.empty(need - 1, dtype=torch.uint8, device=DEV)), old)
    out = torch.empty((B, Cout, 2 * N - n, 2 * N - n), device=DEV)
    kst.kst_forward_seg_static(x, seg, Cout, n, out)
    assert torch.equal(out, kst.kst_forward_seg(x, seg, Cout, n))
