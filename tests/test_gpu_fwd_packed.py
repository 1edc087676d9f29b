"""fp32 forward layers whose input is repacked: against the oracle, bit for bit on integers with guard words around the output,
both forms of the multiply, infinities and NaN, and less scratch."""
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import TOL, check_exact_with_guards, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def repacked_bytes(B, Cin, N, P):
    return B * -(-Cin // 16) * 3 * (N + 2 * ((P + 1) // 2)) ** 2 * 32


# Kernel edges with few and many output channels (rows and classes form), both tile and stage sizes, whole and split
# reductions, ragged channels, odd maps and padding factors.
SHAPES = [
    (5, 26, 288, 40, 5, 0),
    (9, 128, 91, 26, 3, 2),
    (5, 300, 72, 19, 4, 3),
    (64, 33, 40, 13, 3, 1),
    (33, 40, 100, 9, 5, 3),
    (46, 248, 3, 11, 4, 2),
    (20, 261, 3, 26, 5, 1),
    (100, 43, 8, 12, 5, 2),
    (7, 100, 7, 33, 3, 0),
    (2, 200, 6, 60, 4, 1),
    (3, 64, 36, 75, 3, 2),
    (200, 17, 16, 10, 4, 0),
]


def _run(x, seg, Cout, n, P, bias=None, act=kst.KST_ACT_NONE, **kw):
    if bias is None and act == kst.KST_ACT_NONE:
        return kst.kst_forward_seg_padded(x, seg, Cout, n, P, **kw)
    return kst.kst_forward_seg_epilogue(x, seg, Cout, n, bias=bias, act=act, P=P, **kw)


@pytest.mark.parametrize("B,Cin,Cout,N,n,P", SHAPES)
def test_fp32_repacked_input(B, Cin, Cout, N, n, P):
    assert kst.kst_workspace_bytes_padded(B, Cin, Cout, N, n, P, kst.KST_F32) >= repacked_bytes(B, Cin, N, P)
    layer = wl.Layer("fwd_packed", B, Cin, Cout, N, n, "f32", "relu_normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 2600 + N + Cin)
    got = _run(x.to(DEV), kst.kst_segregate_weights(w.to(DEV)), Cout, n, P)
    items = sorted({0, B // 2, B - 1})
    want = oracle.forward(wl.to_f64(x[items]), wl.to_f64(w), P)
    assert rel_err(got[items].cpu().numpy(), want) <= TOL["f32"]
    check_exact_with_guards(wl.Layer("fwd_packed_int", B, Cin, Cout, N, n, "f32", "integer"), kst.KST_PATH_AUTO, 2700 + N, P=P)


@pytest.mark.parametrize("act", [kst.KST_ACT_NONE, kst.KST_ACT_RELU, kst.KST_ACT_TANH])
@pytest.mark.parametrize("B,Cin,Cout,N,n,P", [SHAPES[2], SHAPES[5], SHAPES[9]])
def test_fp32_repacked_input_epilogue(B, Cin, Cout, N, n, P, act):
    layer = wl.Layer("fwd_packed_epi", B, Cin, Cout, N, n, "f32", "relu_normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 2800 + N)
    bias = torch.randn(Cout, generator=torch.Generator().manual_seed(7))
    got = _run(x.to(DEV), kst.kst_segregate_weights(w.to(DEV)), Cout, n, P, bias.to(DEV), act)
    items = sorted({0, B - 1})
    want = oracle.forward_epilogue(wl.to_f64(x[items]), wl.to_f64(w), wl.to_f64(bias), act, P)
    assert rel_err(got[items].cpu().numpy(), want) <= TOL["f32"]


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[6], SHAPES[9]])
def test_fp32_repacked_input_not_finite(shape):
    """Values that are not finite, and finite ones whose scaled parts are not, give what the fp32 multiplies give."""
    B, Cin, Cout, N, n, P = shape
    layer = wl.Layer("fwd_packed_inf", B, Cin, Cout, N, n, "f32", "normal", w_std=0.1)
    x, w = wl.make_tensors(layer, 2900)
    x[0, Cin - 1, N // 2, N // 2] = float("inf")
    x[B - 1, 0, 0, 1] = float("nan")
    x[0, 1, 1, N - 1] = 3.0e38
    w[Cout - 1, 2, 0, n - 1] = 1.0e30
    seg = kst.kst_segregate_weights(w.to(DEV))
    got = _run(x.to(DEV), seg, Cout, n, P)
    old = _run(x.to(DEV), seg, Cout, n, P, path=kst.KST_PATH_IGEMM if Cout >= 16 else kst.KST_PATH_DIRECT)
    finite = torch.isfinite(old)
    assert torch.equal(torch.isfinite(got), finite) and not finite.all() and finite.any()
    assert torch.equal(torch.isnan(got), torch.isnan(old))
    big = old.where(finite, torch.zeros((), device=DEV)).abs()
    near = (got - old).abs() <= 4 * TOL["f32"] * torch.maximum(big, torch.tensor(30.0, device=DEV))
    assert near[finite & (big < 1e6)].all()
    # beside the huge weight a sum's error is that of its largest product
    assert ((got - old).abs() <= 1e-4 * torch.maximum(big, torch.tensor(1e31, device=DEV)))[finite].all()


def test_fp32_less_scratch_than_the_repacked_input():
    for shape in (SHAPES[0], SHAPES[5], SHAPES[10]):
        B, Cin, Cout, N, n, P = shape
        layer = wl.Layer("fwd_packed_ws", B, Cin, Cout, N, n, "f32", "relu_normal", w_std=0.1)
        x, w = wl.make_tensors(layer, 2950)
        x, seg = x.to(DEV), kst.kst_segregate_weights(w.to(DEV))
        dims = (B, Cin, Cout, N, n, P, kst.KST_F32)
        need = kst.kst_workspace_bytes_padded(*dims)
        full, other = _run(x, seg, Cout, n, P), 0
        have = need - 1
        while have > 64:                              # the kernels that do without, as far as it is enough for those
            try:
                less = _run(x, seg, Cout, n, P, ws=torch.empty(have, dtype=torch.uint8, device=DEV))
                assert float((full - less).abs().max()) <= 2 * TOL["f32"] * float(full.abs().max())
                other += not torch.equal(full, less)
            except kst.KstError as e:
                assert e.status == 4                  # KST_ERR_WORKSPACE
                other += 1
            have = have * 7 // 8
        assert other > 0
