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
# Whole batch items and strips, the three shapes of a wave, steps that are no multiple of its segments.
KERNEL_GRADIENT = [
    (64, 512, 256, 8, 4, 2, "f32"), (45, 250, 250, 19, 3, 1, "f32"), (21, 300, 130, 21, 5, 0, "f32"), (96, 64, 250, 13, 5, 2, "f32"), (128, 96, 64, 16, 5, 2, "f32"),
    (64, 256, 128, 16, 4, 2, "f16"), (70, 250, 60, 15, 5, 3, "f16"), (60, 384, 130, 10, 3, 1, "f16"),
]


def _inputs(shape, seed):
    B, Cin, Cout, N, n, P = shape[:6]
    dt = _DT[shape[6]] if len(shape) > 6 else torch.float32
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn((B, Cin, N, N), generator=gen).clamp_(min=0.0).to(dt)
    w = (torch.randn((Cout, Cin, n, n), generator=gen) * 0.05).to(dt)
    M = 2 * N + 2 * P - n
    g = torch.randn((B, Cout, M, M), generator=gen) * 0.1
    for t in (x, w, g):                                           # (one in some tens of these tensors would have three parts)
        t[t.abs() < 1e-6] = 0.0
    return x, w, g


def _forward(x, w, P, path=kst.KST_PATH_AUTO):
    out = kst.kst_forward_seg_padded(x, kst.kst_segregate_weights(w), w.shape[0], w.shape[2], P, path=path)
    torch.cuda.synchronize()
    return out


def _wide(t):
    """The tensor with its last item's first plane 2^-36 and more below its largest value: three parts."""
    t = t.clone()
    t[-1, 0] = 1e-12
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


@pytest.mark.parametrize("shape", KERNEL_GRADIENT)
def test_kernel_gradient(shape):
    B, Cin, Cout, N, n, P, _ = shape
    x, _, g = (t.to(DEV) for t in _inputs(shape, 47 + B))
    low = g.clone()
    low[:, -1] *= 1e-12                                           # (an output channel that the others have no part in)
    dw, three = kst.kst_backward_weight(x, g, n, P), kst.kst_backward_weight(x, low, n, P)
    assert not torch.equal(dw[:-1], three[:-1])
    assert torch.equal(dw, kst.kst_backward_weight(x, g, n, P))
    cos, cis = sorted({0, 31, Cout // 2, Cout - 2}), sorted({0, 33, Cin // 2, Cin - 1})
    want = oracle.backward_weight(wl.to_f64(x[:, cis].cpu()), wl.to_f64(g[:, cos].cpu()), n, P)
    got, other = dw[cos][:, cis], three[cos][:, cis]
    assert np.abs(got.cpu().numpy() - want).max() <= TOL * np.abs(want).max()
    # (a few hundred elements: their errors' scatter is a tenth)
    here, there = _errors(got, other, want)
    assert here <= 1.2 * there, (here, there)
    # every element: one random combination of the input channels
    r = torch.randn(Cin, generator=torch.Generator().manual_seed(4)).double()
    xr = torch.einsum("bihw,i->bhw", x.cpu().double(), r)[:, None].numpy()
    want = oracle.backward_weight(np.ascontiguousarray(xr), wl.to_f64(g.cpu()), n, P)[:, 0]
    mine = (dw.double() * r.to(DEV).view(1, -1, 1, 1)).sum(1).cpu().numpy()
    assert np.abs(mine - want).max() <= TOL * np.abs(want).max()


# Values 2^29 below the largest magnitude still have two parts, with 2^30 below it the tensor has not.
@pytest.mark.parametrize("low", [2.0 ** -12, 2.0 ** -15, 2.0 ** -27, 2.0 ** -29, 2.0 ** -30, 1e-20, 1e-40])
def test_ranges(low):
    shape = (64, 512, 256, 8, 4, 2)
    x, w, g = (t.to(DEV) for t in _inputs(shape, 5))
    N, n, P = 8, 4, 2
    ones = torch.where(g == 0, 1.0, torch.sign(g)) * (1.0 + g.abs() % 1.0)          # magnitudes in [1, 2)
    scaled = ones.clone()
    scaled[1] *= low
    din, ref = kst.kst_backward_input(scaled, w, N, P), kst.kst_backward_input(ones, w, N, P)
    assert torch.equal(din[2:], ref[2:]) == (low >= 2.0 ** -29)   # (other parts, other sums)
    if low >= 2.0 ** -15:                                         # (second parts are normal numbers)
        assert torch.equal(din[1], ref[1] * low)
    want = oracle.backward_input(wl.to_f64(scaled[:2].cpu()), wl.to_f64(w.cpu()), N, P)
    got = din[:2].cpu().numpy().astype(np.float64)
    for i in range(2):
        assert np.abs(got[i] - want[i]).max() <= max(TOL * np.abs(want[i]).max(), 1e-44)
        if low >= 1e-20:
            assert np.linalg.norm(got[i] - want[i]) <= 4e-7 * np.linalg.norm(want[i])


# Tensors of 4 k + 2 values: the last two are no whole load of the ranges' pass; the first and one in the middle beside them.
@pytest.mark.parametrize("at", [0, 2000003, -3, -2, -1])
@pytest.mark.parametrize("which", ["x", "g"])
def test_every_value_is_looked_at(which, at):
    shape = KERNEL_GRADIENT[1]
    x, _, g = (t.to(DEV) for t in _inputs(shape, 14))
    n, P = shape[4:6]
    t = x if which == "x" else g
    assert t.numel() % 4 == 2
    t.view(-1)[at] = 0.0
    two = kst.kst_backward_weight(x, g, n, P)
    t.view(-1)[at] = 1e-20                                        # (below half a last bit of every sum)
    assert not torch.equal(two, kst.kst_backward_weight(x, g, n, P))


# Shares of the products that are not zero well above and well below what a plan wants (forward 32 of 114 steps, input gradient 28 of 56,
# kernel gradients 22 of 56 and 18 of 60): few additions that round are more exact in three parts.
@pytest.mark.parametrize("share,two", [(0.6, True), (0.08, False)])
@pytest.mark.parametrize("name", ["forward", "input", "kernel", "kernel f16", "kernel g"])
def test_zeros_count(name, share, two):
    shape = FORWARD[0] if name == "forward" else KERNEL_GRADIENT[5] if name == "kernel f16" else INPUT_GRADIENT[0]
    x, w, g = (t.to(DEV) for t in _inputs(shape, 12))
    N, n, P = shape[3:6]
    x[x == 0] = 0.5
    sparse = g if name in ("input", "kernel g") else x
    keep = torch.rand(sparse.shape, generator=torch.Generator().manual_seed(13)).to(DEV) < share
    sparse *= keep
    if name == "forward":
        got, three = (_forward(t, w, P)[:-1] for t in (x, _wide(x)))
    elif name == "input":
        got, three = (kst.kst_backward_input(t, w, N, P)[:-1] for t in (g, _wide(g)))
    else:
        low = g.clone()
        low[:, -1] *= 1e-12
        got, three = (kst.kst_backward_weight(x, t, n, P)[:-1] for t in (g, low))
    assert torch.equal(got, three) == (not two)


@pytest.mark.parametrize("low", [2.0 ** -10, 2.0 ** -16, 1e-7, 1e-30])
def test_a_small_channel(low):
    """A channel of the result that is far smaller than the others, by its weights or its share of an operand, maps of 4 x 4
    included: as exact by itself as the whole is."""
    B, Cin, Cout, N, n, P = FORWARD[0]
    x, w, _ = (t.to(DEV) for t in _inputs(FORWARD[0], 8))
    w[37] *= low
    got = _forward(x, w, P)[:2, 37].cpu().numpy().astype(np.float64)
    want = oracle.forward(wl.to_f64(x[:2].cpu()), wl.to_f64(w[37:38].cpu()), P)[:, 0]
    assert np.linalg.norm(got - want) <= 3e-7 * np.linalg.norm(want)
    for shape in ((64, 512, 256, 8, 4, 2), (300, 300, 260, 4, 4, 2)):
        x, w, g = (t.to(DEV) for t in _inputs(shape, 9))
        N, n, P = shape[3:6]
        w[:, 37] *= low
        got = kst.kst_backward_input(g, w, N, P)[:4, 37].cpu().numpy().astype(np.float64)
        want = oracle.backward_input(wl.to_f64(g[:4].cpu()), wl.to_f64(w[:, 37:38].cpu()), N, P)[:, 0]
        assert np.linalg.norm(got - want) <= 4e-7 * np.linalg.norm(want)
        for t, which in ((x, lambda d: d[:64, 37]), (g, lambda d: d[37, :64])):
            keep = t[:, 37].clone()
            t[:, 37] *= low
            got = which(kst.kst_backward_weight(x, g, n, P)).cpu().numpy().astype(np.float64)
            xs, gs = (x[:, 37:38], g[:, :64]) if t is x else (x[:, :64], g[:, 37:38])
            want = oracle.backward_weight(wl.to_f64(xs.cpu()), wl.to_f64(gs.cpu()), n, P)
            want = want[:, 0] if t is x else want[0]
            assert np.linalg.norm(got - want) <= 4e-7 * np.linalg.norm(want)
            t[:, 37] = keep


def test_zeros_and_values_that_are_not_finite():
    shape = (64, 512, 256, 8, 4, 2)
    x, w, g = (t.to(DEV) for t in _inputs(shape, 6))
    N, n, P = 8, 4, 2
    assert not kst.kst_backward_input(torch.zeros_like(g), w, N, P).any()
    assert not kst.kst_backward_weight(x, torch.zeros_like(g), n, P).any()
    for bad in (float("inf"), float("nan")):
        h = g.clone()
        h[3, 2, 8, 8] = bad
        din, ref = kst.kst_backward_input(h, w, N, P), kst.kst_backward_input(g, w, N, P)
        assert not torch.isfinite(din[3]).all() and torch.isfinite(din[:3]).all() and torch.isfinite(din[4:]).all()
        assert float((din[:3] - ref[:3]).abs().max()) <= TOL * float(ref.abs().max())
        half = x.half()
        half[0, 1, 2, 3] = bad
        dw = kst.kst_backward_weight(half, g, n, P)
        assert not torch.isfinite(dw[:, 1]).all() and torch.isfinite(dw[:, 2:]).all()


@pytest.mark.parametrize("name", ["forward", "input", "kernel"])
def test_replayed_graph(name):
    """Captured once, replayed with other inputs of the same and of a wide range, each against the eager call."""
    shape = (31, 600, 200, 16, 4, 0) if name == "forward" else (64, 512, 256, 8, 4, 2)
    B, Cin, Cout, N, n, P = shape
    x, w, g = (t.to(DEV) for t in _inputs(shape, 7))
    dims = (B, Cin, Cout, N, n, P, kst.KST_F32)
    if name == "forward":
        src, out = x, torch.empty((B, Cout, 2 * N + 2 * P - n, 2 * N + 2 * P - n), device=DEV)
        seg, ws = kst.kst_segregate_weights(w), torch.empty(kst.kst_workspace_bytes_padded(*dims), dtype=torch.uint8, device=DEV)
        call = lambda t, o: kst.kst_forward_seg_padded(t, seg, Cout, n, P, out=o, ws=ws)
    elif name == "input":
        src, out = g, torch.empty((B, Cin, N, N), device=DEV)
        ws = torch.empty(kst.kst_backward_input_workspace_bytes(*dims), dtype=torch.uint8, device=DEV)
        call = lambda t, o: kst.kst_backward_input(t, w, N, P, din=o, ws=ws)
    else:
        src, out = g, torch.empty((Cout, Cin, n, n), device=DEV)
        ws = torch.empty(kst.kst_backward_weight_workspace_bytes(*dims), dtype=torch.uint8, device=DEV)
        call = lambda t, o: kst.kst_backward_weight(x, t, n, P, dw=o, ws=ws)
    static = src.clone()
    call(static, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(static, out)
    for t in (src, src * 3.0, _wide(src), src * 2.0 ** 30, src):
        want = call(t, torch.empty_like(out))
        static.copy_(t)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
