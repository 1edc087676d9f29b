"""Gradients of layers with a handful of channels on any map from 32 pixels: strips of every height, rows that are no whole
groups of four, odd padding factors with g as it lies in memory, one workgroup and hundreds."""
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import GRAD_TOL, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}

SHAPES = [
    (1, 1, 1, 32, 3, 0, "f32"),        # the smallest map, strips of two rows
    (1, 3, 1, 33, 5, 1, "f32"),        # odd rows, odd padding factor
    (3, 3, 1, 65, 4, 3, "bf16"),
    (2, 2, 3, 67, 3, 1, "f16"),        # several output channels
    (40, 3, 1, 45, 5, 3, "f32"),       # strips of eight rows, the last one of five
    (9, 4, 2, 70, 5, 2, "f32"),        # 100 sums per lane
    (5, 1, 8, 53, 7, 5, "f32"),        # the largest kernel, padding factor of more than the kernel's reach on one side
    (2, 3, 1, 262, 4, 1, "f32"),       # g wider than a lane's registers hold: staged strip after strip
    (30, 3, 1, 129, 3, 3, "f32"),      # more strips than workgroups
    (1, 4, 1, 36, 1, 0, "f32"),        # one tap
]


def _inputs(B, Cin, Cout, N, n, P, dtype, integer=False):
    layer = wl.Layer("image_grad", B, Cin, Cout, N, n, dtype, "integer" if integer else "normal", w_std=0.2, P=P)
    x, w = wl.make_tensors(layer, 31 + N)
    M = 2 * N + 2 * P - n
    gen = torch.Generator().manual_seed(N + n)
    g = torch.randint(-3, 4, (B, Cout, M, M), generator=gen).float() if integer else torch.randn((B, Cout, M, M), generator=gen)
    return x, w, g


@pytest.mark.parametrize("B,Cin,Cout,N,n,P,dtype", SHAPES)
def test_image_gradients(B, Cin, Cout, N, n, P, dtype):
    x, w, g = _inputs(B, Cin, Cout, N, n, P, dtype)
    # no framed copy of g: the partial results of at most 512 workgroups, and nothing for the input gradient
    dims = (B, Cin, Cout, N, n, P, CODE[dtype])
    assert kst.kst_backward_weight_workspace_bytes(*dims) <= 512 * Cout * Cin * n * n * 4 + 256
    dw = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)
    din = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)
    assert rel_err(dw.cpu().numpy(), oracle.backward_weight(wl.to_f64(x), wl.to_f64(g), n, P)) <= GRAD_TOL[dtype]
    assert rel_err(din.cpu().numpy(), oracle.backward_input(wl.to_f64(g), wl.to_f64(w), N, P)) <= GRAD_TOL[dtype]
    # whole numbers: every order of the sums gives the same
    x, w, g = _inputs(B, Cin, Cout, N, n, P, dtype, integer=True)
    guard = torch.full((Cout * Cin * n * n + 64,), 7.5, device=DEV)
    out = guard[32:-32].view(Cout, Cin, n, n)
    kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P, dw=out)
    want = torch.from_numpy(oracle.backward_weight(wl.to_f64(x), wl.to_f64(g), n, P))
    assert want.abs().max() < 2 ** 24 and torch.equal(out.cpu().double(), want)
    assert (guard[:32] == 7.5).all() and (guard[-32:] == 7.5).all()


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_image_gradients_not_finite(value):
    """A value of g that is not finite reaches the kernel elements it meets an input pixel with, and no others."""
    B, Cin, Cout, N, n, P = 2, 3, 1, 37, 4, 1
    x, w, g = _inputs(B, Cin, Cout, N, n, P, "f32")
    x = x.abs() + 0.5
    g[1, 0, 0, 2] = value                              # row 0: taps u with 2 a + P - u = 0
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P).cpu()
    hit = torch.zeros(n, n, dtype=torch.bool)
    for u in range(n):
        for v in range(n):
            a, c = (0 - P + u), (2 - P + v)
            hit[u, v] = a % 2 == 0 and c % 2 == 0 and 0 <= a // 2 < N and 0 <= c // 2 < N
    assert torch.equal(~torch.isfinite(got), hit.expand(Cout, Cin, n, n)) and hit.any() and not hit.all()
