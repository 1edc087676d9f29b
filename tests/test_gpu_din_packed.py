"""Input gradient with g repacked once: against the oracle, bit for bit on integers with guard words around the result."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl
from test_gpu_parity import GRAD_TOL, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CODE = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}


def repacked_bytes(B, Cout, N, n):
    """g's three parts with the frame the taps reach: sixteen channels of four planes, or four channels' four parities."""
    edge = N + (n - 1) // 2
    return B * (-(-Cout // 4) * 1 if Cout <= 4 else -(-Cout // 16) * 4) * 3 * edge * edge * 32


# Both tile sizes and stage sizes, whole and split reductions, ragged channels, odd maps and padding factors, every type, one
# to four output channels (all parities in one chunk).
SHAPES = [
    (10, 23, 368, 31, 4, 2, "f16"),
    (5, 26, 288, 40, 5, 0, "f32"),
    (7, 73, 52, 29, 4, 2, "f16"),
    (3, 100, 33, 25, 3, 3, "bf16"),
    (1, 70, 200, 27, 5, 1, "f32"),
    (64, 40, 48, 12, 3, 1, "f32"),
    (17, 33, 100, 4, 5, 2, "bf16"),
    (300, 32, 20, 7, 3, 0, "f32"),
    (2, 128, 130, 30, 4, 3, "bf16"),
    (2, 64, 40, 100, 4, 1, "f32"),      # long rows
    (20, 200, 3, 22, 5, 1, "bf16"),     # three output channels
    (33, 64, 3, 32, 4, 2, "f32"),
    (60, 130, 1, 19, 3, 0, "f16"),
    (40, 65, 4, 13, 4, 3, "f32"),
]


def _inputs(B, Cin, Cout, N, n, P, dtype, integer=False):
    layer = wl.Layer("din_packed", B, Cin, Cout, N, n, dtype, "integer" if integer else "normal", w_std=0.2, P=P)
    _, w = wl.make_tensors(layer, 61 + N)
    M = 2 * N + 2 * P - n
    gen = torch.Generator().manual_seed(N + n)
    g = torch.randint(-3, 4, (B, Cout, M, M), generator=gen).float() if integer else torch.randn((B, Cout, M, M), generator=gen)
    return w, g


@pytest.mark.parametrize("B,Cin,Cout,N,n,P,dtype", SHAPES)
def test_input_gradient_of_repacked_g(B, Cin, Cout, N, n, P, dtype):
    assert kst.kst_backward_input_workspace_bytes(B, Cin, Cout, N, n, P, CODE[dtype]) >= repacked_bytes(B, Cout, N, n)
    w, g = _inputs(B, Cin, Cout, N, n, P, dtype)
    din = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)
    assert torch.equal(din, kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P))
    items = sorted({0, B // 2, B - 1})
    want = oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P)
    assert rel_err(din[items].cpu().numpy(), want) <= GRAD_TOL[dtype]
    w, g = _inputs(B, Cin, Cout, N, n, P, dtype, integer=True)
    guard = torch.full((B * Cin * N * N + 64,), 7.5, device=DEV)
    out = guard[32:-32].view(B, Cin, N, N)
    kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P, din=out)
    want = torch.from_numpy(oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P))
    assert want.abs().max() < 2 ** 24 and torch.equal(out[items].cpu().double(), want)
    assert (guard[:32] == 7.5).all() and (guard[-32:] == 7.5).all()


@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[4], SHAPES[10]])
def test_input_gradient_of_repacked_g_not_finite(shape):
    """Infinities, NaN and sums past what the scaled parts hold: where the definition has them, the others untouched."""
    B, Cin, Cout, N, n, P, dtype = shape
    w, g = _inputs(*shape)
    M = g.shape[2]
    g[0, Cout - 1, M // 2, 3] = float("inf")
    g[B - 1, 0, M - 1, M - 1] = float("nan")
    g[0, 0, 1, 1] = 3.0e38                             # (rounds to infinity in no part, its scaled sums do)
    din = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P).cpu()
    items = sorted({0, B - 1})
    with np.errstate(invalid="ignore"):
        want = torch.from_numpy(oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P)).float()
    got, finite = din[items], torch.isfinite(want)
    assert torch.equal(torch.isfinite(got), finite) and torch.equal(torch.isnan(got), torch.isnan(want))
    size = want.where(finite, torch.zeros(())).abs()
    assert ((got - want)[finite].abs() <= GRAD_TOL[dtype] * torch.maximum(size, torch.tensor(30.0))[finite]).all()


def test_less_scratch_than_the_repacked_g():
    for shape in (SHAPES[0], SHAPES[1], SHAPES[11]):
        B, Cin, Cout, N, n, P, dtype = shape
        have = need = kst.kst_backward_input_workspace_bytes(*shape[:6], CODE[dtype])
        w, g = (t.to(DEV) for t in _inputs(*shape))
        full, other = kst.kst_backward_input(g, w, N, P, ws=torch.empty(need, dtype=torch.uint8, device=DEV)), 0
        while have > 64:
            have = have * 7 // 8 // 16 * 16
            try:
                got = kst.kst_backward_input(g, w, N, P, ws=torch.empty(have, dtype=torch.uint8, device=DEV))
                assert float((full - got).abs().max()) <= 2 * GRAD_TOL[dtype] * float(full.abs().max())
                other += 1
            except kst.KstError as e:
                assert e.status == 4                  # KST_ERR_WORKSPACE
                other += 1
        assert other > 0
