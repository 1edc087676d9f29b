"""Kernel gradient of layers with few batch items on the bf16 matrix cores: items cut into strips of rows, every shape of a
wave's tile."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import GRAD_TOL, rel_err
from test_split_plans import split_dw_query

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}

SHAPES = [
    (2, 100, 70, 21, 5, 1, "f32"),      # strips whose last one is short, ragged blocks, odd number of taps
    (4, 49, 32, 30, 4, 2, "f32"),       # one block of output channels: four taps per wave
    (3, 96, 70, 23, 3, 3, "bf16"),      # one block of input channels more than pairs of them
    (5, 65, 200, 17, 4, 1, "f16"),      # two parts of half precision
    (17, 50, 33, 19, 5, 0, "f16"),
    (9, 160, 96, 13, 3, 0, "bf16"),
    (33, 64, 32, 9, 5, 3, "bf16"),      # more items than groups
    (2, 250, 130, 16, 5, 2, "f32"),
    (300, 48, 40, 4, 5, 2, "f32"),      # whole items only
]


def _inputs(B, Cin, Cout, N, n, P, dtype, integer=False):
    layer = wl.Layer("strips", B, Cin, Cout, N, n, dtype, "integer" if integer else "relu_normal", P=P)
    x, _ = wl.make_tensors(layer, 41 + N)
    M = 2 * N + 2 * P - n
    gen = torch.Generator().manual_seed(N + n)
    g = torch.randint(-3, 4, (B, Cout, M, M), generator=gen).float() if integer else torch.randn((B, Cout, M, M), generator=gen)
    return x, g


@pytest.mark.parametrize("B,Cin,Cout,N,n,P,dtype", SHAPES)
def test_kernel_gradient_in_strips(B, Cin, Cout, N, n, P, dtype):
    dims = (B, Cin, Cout, N, n, P, CODE[dtype])
    need = kst.kst_backward_weight_workspace_bytes(*dims)
    assert need != split_dw_query(*dims)
    x, g = _inputs(B, Cin, Cout, N, n, P, dtype)
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)
    assert torch.equal(got, kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P))
    assert rel_err(got.cpu().numpy(), oracle.backward_weight(wl.to_f64(x), wl.to_f64(g), n, P)) <= GRAD_TOL[dtype]
    # whole numbers, exactly, and nothing written beside the result
    x, g = _inputs(B, Cin, Cout, N, n, P, dtype, integer=True)
    guard = torch.full((Cout * Cin * n * n + 64,), 7.5, device=DEV)
    kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P, dw=guard[32:-32].view(Cout, Cin, n, n))
    want = torch.from_numpy(oracle.backward_weight(wl.to_f64(x), wl.to_f64(g), n, P))
    assert want.abs().max() < 2 ** 24 and torch.equal(guard[32:-32].view(want.shape).cpu().double(), want)
    assert (guard[:32] == 7.5).all() and (guard[-32:] == 7.5).all()


def test_kernel_gradient_in_strips_not_finite():
    """Infinities and NaN reach the sums they are in, at a strip's shared rows too."""
    B, Cin, Cout, N, n, P, dtype = SHAPES[0]
    x, g = _inputs(*SHAPES[0])
    x = x + 0.5                                        # (no zeros: every product with an infinity is one)
    M = g.shape[2]
    g[0, 1, M // 2, M // 2] = float("inf")
    g[1, 3, 0, 0] = float("nan")
    x[B - 1, 5, N // 2, N // 2] = float("inf")            # (every tap of it inside the map)
    g = g + (g == 0)
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P).cpu()
    want = torch.zeros((Cout, Cin, n, n), dtype=torch.float64)
    xd, gd = x.double(), g.double()
    for u in range(n):
        for v in range(n):
            rows = [a for a in range(N) if 0 <= 2 * a + P - u < M]
            cols = [c for c in range(N) if 0 <= 2 * c + P - v < M]
            gs = gd[:, :, [2 * a + P - u for a in rows]][:, :, :, [2 * c + P - v for c in cols]]
            xs = xd[:, :, rows][:, :, :, cols]
            want[:, :, u, v] = gs.transpose(0, 1).flatten(1) @ xs.transpose(0, 1).flatten(1).t()
    finite = torch.isfinite(want)
    assert torch.equal(torch.isfinite(got), finite) and torch.equal(torch.isnan(got), torch.isnan(want))
    assert (~finite).any() and finite.any()
    assert ((got.double() - want)[finite].abs() <= GRAD_TOL["f32"] * want[finite].abs().max()).all()


def test_less_scratch_than_the_strips():
    """Less and less scratch: this path, then the kernels that multiply in fp32 as far as it is enough for those, then refused."""
    for shape in (SHAPES[0], SHAPES[5], SHAPES[6]):
        B, Cin, Cout, N, n, P, dtype = shape
        have = need = kst.kst_backward_weight_workspace_bytes(*shape[:6], CODE[dtype])
        x, g = (t.to(DEV) for t in _inputs(*shape))
        full, refused = kst.kst_backward_weight(x, g, n, P, ws=torch.empty(need, dtype=torch.uint8, device=DEV)), 0
        while have > 64:
            have = have * 7 // 8 // 16 * 16
            try:
                got = kst.kst_backward_weight(x, g, n, P, ws=torch.empty(have, dtype=torch.uint8, device=DEV))
                assert float((full - got).abs().max()) <= 2 * GRAD_TOL[dtype] * float(full.abs().max())
            except kst.KstError as e:
                assert e.status == 4                  # KST_ERR_WORKSPACE
                refused += 1
        assert refused > 0
