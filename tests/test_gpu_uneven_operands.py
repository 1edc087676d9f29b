"""Operands of uneven magnitude in large layers: every result as exact as its own operands allow, whatever lies beside it.

A result is a sum of products, so zeros and small values of one operand choose which values of the other count.  Here some
results are made of nothing but small values, next to large ones that they do not see, and are held by themselves against 64
bits: sums of a thousand and more fp32 products of one sign or random ones are within 4e-7 of it in the 2-norm (three bfloat16
parts: 1.2e-7 to 2.5e-7; the same operands alone in their tensor the same)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 4e-7
SCALES = [1e-3, 1e-5, 1e-7, 1e-9, 1e-12, 1e-20]


def _inputs(B, Cin, Cout, N, n, P, seed, relu=True):
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn((B, Cin, N, N), generator=gen)
    if relu:
        x.clamp_(min=0.0)
    w = torch.randn((Cout, Cin, n, n), generator=gen) * 0.05
    M = 2 * N + 2 * P - n
    return x, w, torch.randn((B, Cout, M, M), generator=gen) * 0.1


def _forward(x, w, P):
    w = w.to(DEV)
    out = kst.kst_forward_seg_padded(x.to(DEV), kst.kst_segregate_weights(w), w.shape[0], w.shape[2], P)
    torch.cuda.synchronize()
    return out.cpu()


def _close(got, want):
    got = np.asarray(got, dtype=np.float64)
    assert want.size and np.linalg.norm(want) > 0
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert err <= TOL, err


def _planes(x, w, out, P, co=(0, 7, 33), items=(0, 1)):
    """(got, want) of some planes: the oracle on two items and three output channels."""
    b = [i for i in items for _ in co]
    c = [o for _ in items for o in co]
    return out[b, c].numpy(), oracle.forward_planes(wl.to_f64(x), wl.to_f64(w), b, c, P)


FORWARD = [(31, 600, 200, 16, 4, 0), (64, 1024, 512, 8, 5, 0), (96, 626, 60, 16, 4, 2)]


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("shape", FORWARD)
def test_forward_half_maps(shape, scale):
    """Right half of every map small: the outputs that see nothing else."""
    P, N = shape[5], shape[3]
    x, w, _ = _inputs(*shape, 3)
    x[..., N // 2:] *= scale
    got, want = _planes(x, w, _forward(x, w, P), P)
    _close(got[..., N + P:], want[..., N + P:])
    _close(got, want)


@pytest.mark.parametrize("scale", SCALES)
def test_forward_hot_column(scale):
    """One large column per map, outputs that it does not reach."""
    shape = FORWARD[0]
    x, w, _ = _inputs(*shape, 4)
    small = x * scale
    small[..., 0] = x[..., 0]
    got, want = _planes(small, w, _forward(small, w, 0), 0)
    _close(got[..., 2:], want[..., 2:])


@pytest.mark.parametrize("scale", SCALES)
def test_forward_channels_behind_zero_weights(scale):
    """Small odd channels, the large even ones' weights zero: the whole result (maps of 7 x 7: 64 neighbours are two planes)."""
    x, w, _ = _inputs(128, 1024, 512, 7, 4, 0, 5)
    x[:, 1::2] *= scale
    w[:, 0::2] = 0.0
    _close(*_planes(x, w, _forward(x, w, 0), 0))


@pytest.mark.parametrize("scale", SCALES)
def test_forward_small_subkernel(scale):
    """Weights of one parity class small: the outputs of that parity alone."""
    shape = FORWARD[0]
    x, w, _ = _inputs(*shape, 6)
    w[:, :, 1::2, 1::2] *= scale
    got, want = _planes(x, w, _forward(x, w, 0), 0)
    _close(got[..., 1::2, 1::2], want[..., 1::2, 1::2])


@pytest.mark.parametrize("scale", SCALES)
def test_forward_single_values(scale):
    """One small value alone in an item: its products are the item's whole result."""
    shape = FORWARD[0]
    x, w, _ = _inputs(*shape, 7)
    x[1] = 0.0
    x[1, 3, 5, 6] = scale
    got, want = _planes(x, w, _forward(x, w, 0), 0, items=(1,))
    _close(got, want)


# Weights of a whole number of periods that fit a walk of any number of workgroups, of none, of odd edges; and layer shapes of the timed kind.
INPUT = [(64, 512, 256, 8, 4, 2), (40, 129, 48, 16, 5, 1), (128, 255, 48, 16, 5, 1), (256, 256, 64, 32, 4, 2), (60, 260, 250, 11, 4, 1)]


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("shape", INPUT)
def test_input_gradient_small_channel(shape, scale):
    """An input channel whose weights are small: its gradient alone."""
    N, P = shape[3], shape[5]
    _, w, g = _inputs(*shape, 8)
    w[:, 37] *= scale
    got = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)[:2, 37].cpu()
    _close(got, oracle.backward_input(wl.to_f64(g[:2]), wl.to_f64(w[:, 37:38]), N, P)[:, 0])


@pytest.mark.parametrize("scale", SCALES)
def test_input_gradient_half_maps(scale):
    """Right half of every g small: the gradients that see nothing else."""
    shape = INPUT[0]
    N, P = shape[3], shape[5]
    _, w, g = _inputs(*shape, 9)
    half = g.shape[3] // 2
    g[..., half:] *= scale
    got = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)[:2, :64].cpu()
    want = oracle.backward_input(wl.to_f64(g[:2]), wl.to_f64(w[:, :64].contiguous()), N, P)
    first = (half - P + shape[4] - 1 + 1) // 2                    # 2 c + P - v >= half for every v
    _close(got[..., first:], want[..., first:])
    _close(got, want)


# Whole items and strips, an odd map whose items are no whole groups.
KERNEL = [(64, 512, 256, 8, 4, 2), (45, 250, 250, 19, 3, 1), (60, 301, 300, 5, 5, 3)]


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("shape", KERNEL)
def test_kernel_gradient_items_behind_zeros(shape, scale):
    """Second half of the batch with small inputs, first half with a g of zero: the whole result."""
    B, Cin, Cout, N, n, P = shape
    x, _, g = _inputs(*shape, 10)
    x[B // 2:] *= scale
    g[:B // 2] = 0.0
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)[:40, :40].cpu()
    _close(got, oracle.backward_weight(wl.to_f64(x[:, :40].contiguous()), wl.to_f64(g[:, :40].contiguous()), n, P))


@pytest.mark.parametrize("scale", SCALES)
@pytest.mark.parametrize("shape", KERNEL)
def test_kernel_gradient_small_channel(shape, scale):
    B, Cin, Cout, N, n, P = shape
    x, _, g = _inputs(*shape, 11)
    x[:, 37] *= scale
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)[:64, 37].cpu()
    _close(got, oracle.backward_weight(wl.to_f64(x[:, 37:38].contiguous()), wl.to_f64(g[:, :64].contiguous()), n, P)[:, 0])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("scale", SCALES)
def test_kernel_gradient_half_maps(scale, dtype):
    """g small where the input is not zero."""
    shape = (64, 256, 128, 16, 4, 2)
    B, Cin, Cout, N, n, P = shape
    x, _, g = _inputs(*shape, 12)
    x[..., :N // 2] = 0.0
    g[..., g.shape[3] // 2 - 4:] *= scale
    if dtype == "f16":
        x = x.half()
    got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)[:40, :40].cpu()
    _close(got, oracle.backward_weight(wl.to_f64(x[:, :40].contiguous()), wl.to_f64(g[:, :40].contiguous()), n, P))


def _wide_values(shape, seed):
    """Magnitudes spread evenly over their logarithm, [2^-28, 1]: two parts, with room below."""
    gen = torch.Generator().manual_seed(seed)
    sign = 1.0 - 2.0 * torch.randint(0, 2, shape, generator=gen)
    return sign * torch.exp2(torch.rand(shape, generator=gen) * -28.0)


def _single(got, want):
    """Results that are one product each: within 2^-20 of it."""
    got, want = np.asarray(got, dtype=np.float64), np.asarray(want, dtype=np.float64)
    assert (want != 0).mean() > 0.2
    assert (np.abs(got - want) <= 2.0 ** -20 * np.abs(want)).all()


def test_single_products_forward():
    B, Cin, Cout, N, n, P = FORWARD[0]
    x, w = _wide_values((B, Cin, N, N), 1), _wide_values((Cout, Cin, n, n), 2)
    row = x[1, torch.arange(64) % Cin, (torch.arange(64) // 8) * 2, (torch.arange(64) % 8) * 2].clone()
    x[1] = 0.0                                                    # one value in each block of 2 x 2 pixels: windows that do not meet
    x[1, torch.arange(64) % Cin, (torch.arange(64) // 8) * 2, (torch.arange(64) % 8) * 2] = row
    out, wide = _forward(x, w, P), x.clone()
    wide[-1, 0, 0, 0] = 2.0 ** -40
    assert not torch.equal(out[0], _forward(wide, w, P)[0])       # (three parts there, two here)
    got, want = _planes(x, w, out, P, co=(0, 7, 33, 150), items=(1,))
    _single(got, want)


def test_single_products_input_gradient():
    B, Cin, Cout, N, n, P = shape = INPUT[0]
    M = 2 * N + 2 * P - n
    w, g = _wide_values((Cout, Cin, n, n), 3), _wide_values((B, Cout, M, M), 4)
    keep = g[1, 5, ::4, ::4].clone()
    g[1] = 0.0
    g[1, 5, ::4, ::4] = keep                                      # at most one tap of a position meets one of them
    din, wide = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P), g.clone()
    wide[-1, 0, 0, 0] = 2.0 ** -40
    assert not torch.equal(din[0], kst.kst_backward_input(wide.to(DEV), w.to(DEV), N, P)[0])
    got = din[1:2].cpu()
    _single(got, oracle.backward_input(wl.to_f64(g[1:2]), wl.to_f64(w), N, P))


def test_single_products_kernel_gradient():
    B, Cin, Cout, N, n, P = KERNEL[0]
    M = 2 * N + 2 * P - n
    x, g = _wide_values((B, Cin, N, N), 5), _wide_values((B, Cout, M, M), 6)
    at = torch.arange(32)
    keep = x[at, at, at % N, at // 4].clone()
    x[:, :32] = 0.0
    x[at, at, at % N, at // 4] = keep                             # one value of each of 32 input channels
    dw, wide = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P), g.clone()
    wide[0, -1, 0, 0] = 2.0 ** -40
    assert not torch.equal(dw[:-1], kst.kst_backward_weight(x.to(DEV), wide.to(DEV), n, P)[:-1])
    got = dw[:40, :32].cpu()
    _single(got, oracle.backward_weight(wl.to_f64(x[:, :32].contiguous()), wl.to_f64(g[:, :40].contiguous()), n, P))
