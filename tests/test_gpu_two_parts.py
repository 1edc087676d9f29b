"""Large layers whose operands are split into two half-precision parts: against the oracle, against the three parts that
tensors of a wide range take, and no less exact than those."""
import numpy as np
import pytest
import torch

import oracle
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 2e-5          # of the largest element, as for every fp32 kernel
_DT = {"f32": torch.float32, "f16": torch.float16}

# Tiles of 128 and 64 output channels, three and five staged positions, an odd number of channel chunks and a last one of two
# channels, odd padding factors, whole and shared passes.
FORWARD = [
    (31, 600, 200, 16, 4, 0), (34, 1010, 130, 13, 4, 1), (96, 626, 60, 16, 4, 2), (9, 500, 130, 45, 4, 0), (20, 530, 64, 40, 4, 3),
    (120, 546, 256, 9, 5, 0), (36, 490, 130, 16, 5, 1), (84, 530, 50, 18, 5, 2), (7, 450, 64, 61, 5, 2),
]
# 128 and 256 input channels per tile, five and seven staged cells, ragged channels.
INPUT_GRADIENT = [
    (64, 512, 256, 8, 4, 2, "f32"), (60, 260, 250, 11, 4, 1, "f32"), (25, 110, 300, 16, 4, 0, "f32"), (28, 100, 290, 14, 4, 3, "f16"),
    (40, 128, 130, 16, 5, 1, "f32"), (190, 130, 90, 8, 5, 2, "f16"),
]


def _inputs(shape, seed):
    B, Cin, Cout, N, n, P = shape[:6]
    dt = _DT[shape[6]] if len(shape) > 6 else torch.float32
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn((B, Cin, N, N), generator=gen).clamp_(min=0.0).to(dt)
    w = (torch.randn((Cout, Cin, n, n), generator=gen) * 0.05).to(dt)
    M = 2 * N + 2 * P - n
    return x, w, torch.randn((B, Cout, M, M), generator=gen) * 0.1


def _forward(x, w, P, path=kst.KST_PATH_AUTO):
    out = kst.kst_forward_seg_padded(x, kst.kst_segregate_weights(w), w.shape[0], w.shape[2], P, path=path)
    torch.cuda.synchronize()
    return out


def _wide(t):
    """The tensor with its last item's first 64 and more values far below all others: three parts."""
    t = t.clone()
    t[-1, 0] = 1e-7
    return t


def _errors(got, other, want):
    return (np.linalg.norm(v.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want) for v in (got, other))


@pytest.mark.parametrize("shape", FORWARD)
def test_forward(shape):
    P = shape[5]
    x, w, _ = (t.to(DEV) for t in _inputs(shape, 31 + shape[0]))
    out, three = _forward(x, w, P), _forward(_wide(x), w, P)
    assert not torch.equal(out[:-1], three[:-1])                  # (other parts, other sums)
    assert torch.equal(out, _forward(x, w, P))
    b, co = [0, 1, 3, x.shape[0] - 2] * 3, [(i * 13 + 5) % w.shape[0] for i in range(11)] + [w.shape[0] - 1]
    want = oracle.forward_planes(wl.to_f64(x.cpu()), wl.to_f64(w.cpu()), b, co, P)
    at = (torch.tensor(b), torch.tensor(co))
    got, other = out.cpu()[at], three.cpu()[at]
    assert np.abs(got.numpy() - want).max() <= TOL * np.abs(want).max()
    here, there = _errors(got, other, want)
    assert here <= 1.03 * there, (here, there)                   # (of some ten thousand elements: within their scatter)
    # every element, against the kernels that multiply in fp32 (1e-6 of a chain of a few thousand roundings on both sides)
    plain = _forward(x, w, P, kst.KST_PATH_IGEMM)
    assert float((out - plain).abs().max()) <= 2 * TOL * float(plain.abs().max())


@pytest.mark.parametrize("shape", INPUT_GRADIENT)
def test_input_gradient(shape):
    N, P = shape[3], shape[5]
    _, w, g = (t.to(DEV) for t in _inputs(shape, 17 + shape[0]))
    din, three = kst.kst_backward_input(g, w, N, P), kst.kst_backward_input(_wide(g), w, N, P)
    assert not torch.equal(din[:-1], three[:-1])
    assert torch.equal(din, kst.kst_backward_input(g, w, N, P))
    items = [0, 1, g.shape[0] // 2, g.shape[0] - 2]
    want = oracle.backward_input(wl.to_f64(g[items].cpu()), wl.to_f64(w.cpu()), N, P)
    assert np.abs(din[items].cpu().numpy() - want).max() <= TOL * np.abs(want).max()
    here, there = _errors(din[items], three[items], want)
    assert here <= 1.03 * there, (here, there)


# A block of 64 neighbours 2^13 below the largest magnitude still has two parts, 2^15 below it has not; what lies beside a
# value far above everything else, or in a channel far below, is as exact as if it were alone.
@pytest.mark.parametrize("low", [2.0 ** -12, 2.0 ** -15, 1e-20, 1e-40])
def test_ranges(low):
    shape = (64, 512, 256, 8, 4, 2)
    x, w, g = (t.to(DEV) for t in _inputs(shape, 5))
    N, n, P = 8, 4, 2
    ones = torch.where(g == 0, 1.0, torch.sign(g)) * (1.0 + g.abs() % 1.0)          # magnitudes in [1, 2)
    scaled = ones.clone()
    scaled[1] *= low
    din, ref = kst.kst_backward_input(scaled, w, N, P), kst.kst_backward_input(ones, w, N, P)
    if low == 2.0 ** -12:
        assert torch.equal(din[1], ref[1] * low) and torch.equal(din[2:], ref[2:])
    want = oracle.backward_input(wl.to_f64(scaled[:2].cpu()), wl.to_f64(w.cpu()), N, P)
    got = din[:2].cpu().numpy().astype(np.float64)
    for i in range(2):
        assert np.abs(got[i] - want[i]).max() <= max(TOL * np.abs(want[i]).max(), 1e-44)
