"""fp32 layers whose operands are split into three bfloat16 parts for the matrix cores: against the oracle and against
the kernels that multiply in fp32."""
import numpy as np
import pytest
import torch

import oracle
import test_split_plans as plans
from paper_2209_03704_amd import binding as kst
from paper_2209_03704_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 2e-5          # of the largest element, as for every fp32 kernel

# Layers the split kernels take (each test asserts it by the workspace; test_split_plans.py holds the lists against every
# variant there is): kernel edges 3, 4, 5; tiles of 64 and 128 output channels; three and five staged positions per lane;
# ragged channels, chunks, batches; odd maps; odd padding factors.
FORWARD = [
    (30, 130, 200, 16, 4, 0),    # ragged channels on both sides, even map
    (26, 515, 66, 13, 3, 2),     # odd map edge and padding, a last chunk of three channels, 66 of 128 channels
    (70, 33, 40, 33, 5, 1),      # tiles of 64 channels, odd padding factor (interior stores), two chunks and one channel
    (9, 96, 130, 64, 3, 0),      # rows of half a tile
    (64, 512, 256, 8, 4, 2),     # shared passes only
    (130, 256, 64, 6, 5, 3),     # small maps, many items per tile, odd padding factor
    (2, 90, 130, 100, 3, 0),     # long rows: five staged positions per lane with tiles of 128 positions
    (2, 70, 130, 90, 4, 0),
    (3, 66, 130, 64, 5, 0),
    (14, 130, 200, 16, 5, 0),
    (250, 65, 48, 16, 3, 0),     # tiles of 64 channels and 256 positions, five and three staged positions
    (25, 90, 50, 40, 3, 0),
    (60, 131, 52, 20, 4, 0),
    (60, 131, 52, 16, 4, 1),
    (40, 130, 50, 18, 5, 0),
]


def _layer(shape, seed):
    B, Cin, Cout, N, n, P = shape
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn((B, Cin, N, N), generator=gen).clamp_(min=0.0)
    w = torch.randn((Cout, Cin, n, n), generator=gen) * 0.05
    return x, w


def _forward(x, w, P, path=kst.KST_PATH_AUTO, bias=None, act=kst.KST_ACT_NONE):
    Cout, n = w.shape[0], w.shape[2]
    wd = kst.kst_segregate_weights(w.to(DEV))
    if bias is not None or act != kst.KST_ACT_NONE:
        out = kst.kst_forward_seg_epilogue(x.to(DEV), wd, Cout, n, bias=None if bias is None else bias.to(DEV), act=act, P=P,
                                           path=path)
    else:
        out = kst.kst_forward_seg_padded(x.to(DEV), wd, Cout, n, P, path=path)
    torch.cuda.synchronize()
    return out.cpu()


def _planes(x, w, P, count=24):
    B, Cout = x.shape[0], w.shape[0]
    b = [(i * 7) % B for i in range(count)] + [B - 1]
    co = [(i * 13 + 5) % Cout for i in range(count)] + [Cout - 1]
    return b, co, oracle.forward_planes(wl.to_f64(x), wl.to_f64(w), b, co, P)


@pytest.mark.parametrize("shape", FORWARD)
def test_split_forward(shape):
    P = shape[5]
    assert kst.kst_workspace_bytes_padded(*shape, kst.KST_F32) == plans.split_forward_bytes(*shape)
    x, w = _layer(shape, 31 + shape[0])
    b, co, want = _planes(x, w, P)
    out = _forward(x, w, P)
    got = out[torch.tensor(b), torch.tensor(co)].numpy().astype(np.float64)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    # every element: a random projection of the channels (the operation is linear in the kernel)
    r = np.random.default_rng(5).standard_normal(w.shape[0])
    proj = oracle.forward(wl.to_f64(x[:2]), np.einsum("o,oiuv->iuv", r, wl.to_f64(w))[None], P)[:, 0]
    mine = np.einsum("o,boyx->byx", r, out[:2].numpy().astype(np.float64))
    assert np.abs(mine - proj).max() <= TOL * np.abs(proj).max()
    # no less precise than fp32 multiplies: the plain kernels, one fp32 multiply-add per product
    plain = _forward(x, w, P, kst.KST_PATH_DIRECT)[torch.tensor(b), torch.tensor(co)].numpy().astype(np.float64)
    assert np.linalg.norm(got - want) <= np.linalg.norm(plain - want)
    assert torch.equal(out, _forward(x, w, P))                    # fixed summing order


@pytest.mark.parametrize("shape", FORWARD[:3])
@pytest.mark.parametrize("act", [kst.KST_ACT_RELU, kst.KST_ACT_TANH])
def test_split_forward_epilogue(shape, act):
    P = shape[5]
    x, w = _layer(shape, 61 + shape[0])
    bias = torch.randn(shape[2], generator=torch.Generator().manual_seed(3))
    bare = _forward(x, w, P).double() + bias.double().view(1, -1, 1, 1)
    want = bare.clamp_(min=0.0) if act == kst.KST_ACT_RELU else torch.tanh(bare)
    got = _forward(x, w, P, bias=bias, act=act).double()
    # one fp32 addition and one tanh (2 ulp) away from the same sums
    assert (got - want).abs().max() <= 1e-6 * max(1.0, float(want.abs().max()))


@pytest.mark.parametrize("shape", [FORWARD[0], FORWARD[2], FORWARD[4]])
def test_split_forward_infinities_and_nan(shape):
    """An infinity, a NaN or a value that bfloat16 rounds to infinity has no three parts: the elements it reaches are
    what fp32 multiplies make of them, all others are untouched."""
    B, Cin, Cout, N, n, P = shape
    x, w = _layer(shape, 91 + B)
    x[0, 1, 2, 3] = float("inf")
    x[B - 1, Cin - 1, N - 1, 0] = float("nan")
    x[B // 2, 0, 0, 0] = 3.4e38
    w[Cout - 1, 3, n - 1, 1] = -float("inf")
    out, ref = _forward(x, w, P), _forward(x, w, P, kst.KST_PATH_DIRECT)
    assert torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(torch.isinf(out), torch.isinf(ref))
    assert torch.equal(out[torch.isinf(out)], ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    item = ref.where(ok, 0.0).abs().amax(dim=(1, 2, 3), keepdim=True).expand_as(ref)   # (one item holds 1e37s)
    assert ((out - ref)[ok].abs() <= TOL * item[ok]).all()


@pytest.mark.parametrize("shape", [FORWARD[0], FORWARD[4]])       # whole passes, shared passes
@pytest.mark.parametrize("act", [kst.KST_ACT_RELU, kst.KST_ACT_TANH])
def test_split_forward_infinities_through_the_epilogue(shape, act):
    B, Cin, Cout, N, n, P = shape
    x, w = _layer(shape, 37 + B)
    x[1, 2, 3, 1] = float("inf")
    x[B - 1, Cin - 1, 0, N - 1] = float("nan")
    x[0] = 2e36 * torch.sign(x[0])                    # a whole item without three parts, its sums well below infinity
    bias = torch.randn(Cout, generator=torch.Generator().manual_seed(3))
    out, ref = (_forward(x, w, P, path, bias=bias, act=act) for path in (kst.KST_PATH_AUTO, kst.KST_PATH_DIRECT))
    assert torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(torch.isinf(out), torch.isinf(ref))
    ok = torch.isfinite(ref)
    scale = 1.0 if act == kst.KST_ACT_TANH else ref.where(ok, 0.0).abs().amax(dim=(1, 2, 3), keepdim=True).expand_as(ref)[ok]
    assert ((out - ref)[ok].abs() <= TOL * scale).all()


def _microseconds(call, count=5):
    call()
    first, last = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    first.record()
    for _ in range(count):
        call()
    last.record()
    torch.cuda.synchronize()
    return first.elapsed_time(last) / count * 1e3


def test_split_one_infinity_stays_affordable():
    """An overflowed value is an ordinary event in training: the elements it reaches are done again a block per wave.
    Measured 3 to 9 times the time without one; one lane per element took 60 to 110 times."""
    B, Cin, Cout, N, n, P = FORWARD[4]
    x, w = (t.to(DEV) for t in _layer(FORWARD[4], 11))
    g = torch.randn((B, Cout, 2 * N + 2 * P - n, 2 * N + 2 * P - n), generator=torch.Generator().manual_seed(12)).to(DEV)
    x_inf, g_inf, seg = x.clone(), g.clone(), kst.kst_segregate_weights(w)
    x_inf[1, 3, 2, 2] = float("inf")
    g_inf[1, 3, N, N] = float("inf")
    for what, call in (("forward", lambda inf: kst.kst_forward_seg_padded(x_inf if inf else x, seg, Cout, n, P)),
                       ("input gradient", lambda inf: kst.kst_backward_input(g_inf if inf else g, w, N, P)),
                       ("kernel gradient", lambda inf: kst.kst_backward_weight(x, g_inf if inf else g, n, P))):
        plain, one = _microseconds(lambda: call(False)), _microseconds(lambda: call(True))
        assert one <= 30 * plain, "%s: %.0f us with one infinity, %.0f without" % (what, one, plain)


# Operand sizes from fp32's smallest to what bfloat16 parts leave room for: exponents of (input or g, weights or input).
SIZES = [(-60, -40), (-126, 60), (70, -126), (-75, -25), (-126, 20), (60, -60)]


def _normal_sized(t, exponent):
    """Values of t's signs in [1, 2) * 2^exponent, zeros kept: scaling by powers of two never rounds them."""
    return torch.where(t == 0, t, torch.copysign(1.0 + (t.abs() % 1.0), t)) * 2.0 ** exponent


@pytest.mark.parametrize("a,b", SIZES)
def test_split_forward_operand_sizes(a, b):
    """Scaling the operands by powers of two scales the result exactly, down to the smallest normal operands."""
    x, w = _layer(FORWARD[4], 7)
    x, w = _normal_sized(x, 0), _normal_sized(w, 0)
    one = _forward(x, w, 2)
    assert torch.equal(_forward(x * 2.0 ** a, w * 2.0 ** b, 2), one * 2.0 ** (a + b))


def test_split_forward_subnormal_operands():
    x, w = _layer(FORWARD[4], 8)
    x = torch.round(x * 2.0 ** 12)                    # whole numbers, so that 2^-149 times them is exact
    one = _forward(x, w, 2)
    tiny = x.double().mul(2.0 ** -149).float()
    assert 0 < tiny[tiny != 0].abs().max() < 2.0 ** -126
    assert torch.equal(_forward(tiny, w * 2.0 ** 100, 2), (one.double() * 2.0 ** -49).float())


# Input gradient: 128 and 256 input channels per tile, five and seven staged cells per lane, ragged channels, odd padding
# factors, tiles that cross items and rows, bfloat16 weights (one part) and half-precision ones (widened).  The first are
# also used below.
INPUT_GRADIENT = [
    (64, 512, 256, 8, 4, 2, "f32"),
    (25, 200, 133, 16, 4, 1, "f32"),
    (17, 130, 70, 33, 3, 0, "f32"),
    (25, 70, 133, 16, 5, 3, "f32"),
    (90, 130, 66, 8, 5, 2, "f32"),
    (9, 96, 130, 64, 3, 2, "f32"),
    (64, 256, 128, 16, 4, 2, "bf16"),
    (40, 70, 130, 21, 3, 1, "bf16"),
    (64, 200, 67, 13, 4, 1, "f16"),
    (10, 60, 90, 32, 5, 1, "f32"),
    (60, 100, 130, 16, 3, 1, "f32"),
    (20, 120, 100, 32, 3, 0, "bf16"),
    (32, 300, 130, 16, 3, 0, "f32"),
    (40, 260, 150, 14, 3, 1, "f32"),
    (130, 258, 140, 8, 3, 2, "bf16"),
    (60, 257, 129, 12, 3, 3, "bf16"),
    (30, 96, 150, 16, 4, 3, "bf16"),
    (56, 128, 90, 15, 4, 1, "bf16"),
    (32, 260, 130, 16, 4, 0, "f32"),
    (70, 260, 130, 11, 4, 2, "bf16"),
    (190, 128, 60, 8, 5, 0, "bf16"),
]
_DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _gradient_inputs(shape, seed):
    B, Cin, Cout, N, n, P, dtype = shape
    x, w = _layer(shape[:6], seed)
    M = 2 * N + 2 * P - n
    g = torch.randn((B, Cout, M, M), generator=torch.Generator().manual_seed(seed + 1)) * 0.1
    return x.to(_DT[dtype]), w.to(_DT[dtype]), g


def _items(B):
    return sorted({0, 1, B // 2, B - 1})


@pytest.mark.parametrize("shape", INPUT_GRADIENT)
def test_split_input_gradient(shape):
    B, Cin, Cout, N, n, P, dtype = shape
    code = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}[dtype]
    assert kst.kst_backward_input_workspace_bytes(*shape[:6], code) == plans.split_din_query(*shape[:6], code)
    _, w, g = _gradient_inputs(shape, 17 + B)
    din = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)
    again = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)
    items = _items(B)
    want = oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P)
    got = din[items].cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    assert torch.equal(din, again)
    # every element: the sum over the input channels with random weights, in fp32 on the GPU against a one-channel layer
    r = torch.randn(Cin, generator=torch.Generator().manual_seed(2)).double()
    wr = torch.einsum("oiuv,i->ouv", w.double(), r)[:, None]
    want = oracle.backward_input(wl.to_f64(g), np.ascontiguousarray(wr.numpy()), N, P)[:, 0]
    got = (din.double() * r.to(DEV).view(1, -1, 1, 1)).sum(1).cpu().numpy()
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("shape", [INPUT_GRADIENT[1], INPUT_GRADIENT[7]])
def test_split_input_gradient_infinities_and_nan(shape):
    B, Cin, Cout, N, n, P, dtype = shape
    _, w, g = _gradient_inputs(shape, 23)
    M = g.shape[2]
    g[0, 1, 2, 3] = float("inf")
    g[B - 1, Cout - 1, M - 1, M - 1] = float("nan")
    w[2, 1, 0, n - 1] = 3.38e38                       # finite in bfloat16 too
    din = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P).cpu()
    items = _items(B)
    with np.errstate(invalid="ignore"):
        want = torch.from_numpy(oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P)).float()
    got = din[items]
    finite = torch.isfinite(want)
    assert torch.equal(torch.isfinite(got), finite)
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    largest = want.where(finite, 0.0).abs().amax(dim=(0, 2, 3), keepdim=True).expand_as(want)   # (one channel holds 1e37s)
    assert ((got - want)[finite].abs() <= TOL * largest[finite]).all()


# Kernel gradient: ragged channel blocks and items, odd numbers of taps, odd padding factors, one and three parts of the
# input, more and fewer splits than steps allow.
KERNEL_GRADIENT = [
    (64, 512, 256, 8, 4, 2, "f32"),
    (30, 250, 127, 19, 3, 1, "f32"),
    (70, 128, 120, 11, 5, 3, "f32"),
    (160, 384, 384, 4, 4, 0, "f32"),
    (64, 256, 128, 16, 4, 2, "bf16"),
    (31, 125, 256, 20, 3, 0, "bf16"),
    (47, 128, 256, 14, 4, 1, "f16"),
    (40, 256, 128, 10, 5, 1, "bf16"),
    (48, 256, 250, 12, 3, 0, "f16"),
    (32, 128, 256, 13, 5, 2, "f16"),
]


@pytest.mark.parametrize("shape", KERNEL_GRADIENT)
def test_split_kernel_gradient(shape):
    B, Cin, Cout, N, n, P, dtype = shape
    code = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}[dtype]
    assert kst.kst_backward_weight_workspace_bytes(*shape[:6], code) == plans.split_dw_query(*shape[:6], code)
    x, _, g = _gradient_inputs(shape, 47 + B)
    dw = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)
    again = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)
    assert torch.equal(dw, again)
    # a few channels of either kind exactly as the oracle has them
    cos, cis = sorted({0, 31, Cout // 2, Cout - 1}), sorted({0, 33, Cin // 2, Cin - 1})
    want = oracle.backward_weight(wl.to_f64(x[:, cis]), wl.to_f64(g[:, cos]), n, P)
    got = dw[cos][:, cis].cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    # every element: random combinations of the channels on one side
    r = torch.randn(Cin, generator=torch.Generator().manual_seed(4)).double()
    xr = torch.einsum("bihw,i->bhw", x.double(), r)[:, None].numpy()
    want = oracle.backward_weight(np.ascontiguousarray(xr), wl.to_f64(g), n, P)[:, 0]
    got = (dw.double() * r.to(DEV).view(1, -1, 1, 1)).sum(1).cpu().numpy()
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()


@pytest.mark.parametrize("shape", [KERNEL_GRADIENT[1], KERNEL_GRADIENT[5]])
def test_split_kernel_gradient_infinities_and_nan(shape):
    B, Cin, Cout, N, n, P, dtype = shape
    x, _, g = _gradient_inputs(shape, 53)
    M = g.shape[2]
    g[0, 1, M // 2, M // 2] = float("inf")
    g[1, 2, M // 2, 3] = 3.4e38
    x[B - 1, 5, N // 2, N // 2] = float("nan")
    x = x.clone()
    x[0, 7] = 1.0                                     # (every product with the infinity is one)
    dw = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P).cpu()
    cos, cis = [0, 1, 2, Cout - 1], [0, 5, 7, Cin - 1]
    # (the oracle multiplies the embedded zeros too, which makes NaN of infinities; here only the terms that exist)
    xd, gd = x[:, cis].double(), g[:, cos].double()
    want = torch.zeros((len(cos), len(cis), n, n), dtype=torch.float64)
    for u in range(n):
        for v in range(n):
            rows = [a for a in range(N) if 0 <= 2 * a + P - u < M]
            cols = [c for c in range(N) if 0 <= 2 * c + P - v < M]
            gs = gd[:, :, [2 * a + P - u for a in rows]][:, :, :, [2 * c + P - v for c in cols]]
            xs = xd[:, :, rows][:, :, :, cols]
            want[:, :, u, v] = (gs[:, :, None] * xs[:, None]).sum(dim=(0, 3, 4))
    want = want.float()
    got = dw[cos][:, cis]
    finite = torch.isfinite(want)
    assert torch.equal(torch.isfinite(got), finite)
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    largest = want.where(finite, 0.0).abs().amax(dim=(1, 2, 3), keepdim=True).expand_as(want)
    assert ((got - want)[finite].abs() <= TOL * largest[finite]).all()


@pytest.mark.parametrize("a,b", SIZES)
def test_split_gradient_operand_sizes(a, b):
    x, w, g = _gradient_inputs(INPUT_GRADIENT[0], 9)
    x, w, g = (_normal_sized(t, 0).to(DEV) for t in (x, w, g))
    N, n, P = x.shape[2], w.shape[2], INPUT_GRADIENT[0][5]
    s, t = 2.0 ** a, 2.0 ** b
    din, dw = kst.kst_backward_input(g, w, N, P), kst.kst_backward_weight(x, g, n, P)
    assert torch.equal(kst.kst_backward_input(g * s, w * t, N, P), din * 2.0 ** (a + b))
    assert torch.equal(kst.kst_backward_weight(x * t, g * s, n, P), dw * 2.0 ** (a + b))


@pytest.mark.parametrize("exponent", [-126, -133])
def test_split_gradients_small_bf16_operands(exponent):
    """bfloat16 operands at and below the smallest normal number (there: whole multiples of 2^-133)."""
    x, w, g = _gradient_inputs(INPUT_GRADIENT[6], 10)
    N, n, P = x.shape[2], w.shape[2], INPUT_GRADIENT[6][5]
    x, w, g = (torch.round(t.float() * 16).to(DEV) for t in (x, w, g * 10))
    small = lambda t: t.double().mul(2.0 ** exponent).to(torch.bfloat16)
    assert torch.equal(small(x).double() * 2.0 ** -exponent, x.double())
    din, dw = kst.kst_backward_input(g, w.bfloat16(), N, P), kst.kst_backward_weight(x.bfloat16(), g, n, P)
    big = g * 2.0 ** 60
    assert torch.equal(kst.kst_backward_input(big, small(w), N, P), din * 2.0 ** (60 + exponent))
    assert torch.equal(kst.kst_backward_weight(small(x), big, n, P), dw * 2.0 ** (60 + exponent))


# Layers just outside the rules (fewer products; maps whose rows of g the input gradient cannot stage): the kernels that
# multiply in fp32, to the same tolerance.
BESIDE = [(23, 515, 66, 13, 3, 2), (30, 128, 66, 19, 5, 3), (33, 40, 530, 10, 5, 2), (45, 128, 120, 11, 5, 3)]


@pytest.mark.parametrize("shape,pass_", zip(BESIDE, ("forward", "input", "input", "kernel")))
def test_layers_beside_the_rules(shape, pass_):
    B, Cin, Cout, N, n, P = shape
    x, w, g = _gradient_inputs((*shape, "f32"), 83)
    if pass_ == "forward":
        assert kst.kst_workspace_bytes_padded(*shape, kst.KST_F32) != plans.split_forward_bytes(*shape)
        b, co, want = _planes(x, w, P)
        got = _forward(x, w, P)[torch.tensor(b), torch.tensor(co)]
    elif pass_ == "input":
        assert kst.kst_backward_input_workspace_bytes(*shape, kst.KST_F32) != plans.split_din_query(*shape, kst.KST_F32)
        items = _items(B)
        want = oracle.backward_input(wl.to_f64(g[items]), wl.to_f64(w), N, P)
        got = kst.kst_backward_input(g.to(DEV), w.to(DEV), N, P)[items].cpu()
    else:
        assert kst.kst_backward_weight_workspace_bytes(*shape, kst.KST_F32) != plans.split_dw_query(*shape, kst.KST_F32)
        cos, cis = [0, 31, Cout - 1], [0, 33, Cin - 1]
        want = oracle.backward_weight(wl.to_f64(x[:, cis]), wl.to_f64(g[:, cos]), n, P)
        got = kst.kst_backward_weight(x.to(DEV), g.to(DEV), n, P)[cos][:, cis].cpu()
    assert np.abs(got.numpy().astype(np.float64) - want).max() <= TOL * np.abs(want).max()


# ---- scratch: what these layers run on with less than they want ------------------------------------------------------

def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None


@pytest.mark.parametrize("shape", [FORWARD[0], FORWARD[4], (64, 1024, 512, 8, 5, 0), (128, 512, 256, 16, 4, 0)])
def test_split_forward_with_less_scratch(shape):
    """A byte less than the split kernels lay out: the kernels that multiply in fp32, bit for bit, where that is enough
    for those; refused where it is not."""
    B, Cin, Cout, N, n, P = shape
    x, w = (t.to(DEV) for t in _layer(shape, 71))
    seg = kst.kst_segregate_weights(w)
    dims = (B, Cin, Cout, N, n, P, kst.KST_F32)
    want, least = kst.kst_workspace_bytes_padded(*dims), kst.kst_workspace_bytes_padded(*dims, kst.KST_PATH_IGEMM)
    call = lambda nbytes, path=kst.KST_PATH_AUTO: kst.kst_forward_seg_padded(x, seg, Cout, n, P, ws=_scratch(nbytes), path=path)
    fp32, split = call(least, kst.KST_PATH_IGEMM), call(want)
    assert not torch.equal(fp32, split)
    assert float((fp32 - split).abs().max()) <= 2 * TOL * float(fp32.abs().max())
    if least < want:
        for have in {least, want - 1}:
            assert torch.equal(call(have) if have else _null_workspace(x, seg, Cout, n, P), fp32)
    if least > 0:                                     # (it may also be the larger of the two)
        with pytest.raises(kst.KstError) as e:
            call(min(least, want) - 1)
        assert e.value.status == 4                    # KST_ERR_WORKSPACE


def _null_workspace(x, seg, Cout, n, P):
    B, Cin, N, _ = x.shape
    out = torch.empty((B, Cout, 2 * N + 2 * P - n, 2 * N + 2 * P - n), device=DEV)
    assert kst.lib().kst_forward_seg_padded(x.data_ptr(), seg.data_ptr(), out.data_ptr(), None, 0, B, Cin, Cout, N, n, P,
                                            kst.KST_F32, kst.KST_PATH_AUTO, torch.cuda.current_stream().cuda_stream) == 0
    return out


def test_split_forward_without_scratch():
    """A layer whose fp32 kernels need no workspace takes a null one."""
    shape = FORWARD[3]
    B, Cin, Cout, N, n, P = shape
    assert kst.kst_workspace_bytes(B, Cin, Cout, N, n, kst.KST_F32, kst.KST_PATH_IGEMM) == 0
    x, w = (t.to(DEV) for t in _layer(shape, 72))
    seg = kst.kst_segregate_weights(w)
    assert torch.equal(_null_workspace(x, seg, Cout, n, P), kst.kst_forward_seg(x, seg, Cout, n, path=kst.KST_PATH_IGEMM))


@pytest.mark.parametrize("shape", [INPUT_GRADIENT[0], INPUT_GRADIENT[6], INPUT_GRADIENT[8]])
def test_split_gradients_with_less_scratch(shape):
    """Every type: with what the query gives, the split kernels; with too little for those, the ones that multiply in
    fp32; a single byte is refused by both."""
    B, Cin, Cout, N, n, P, dtype = shape
    x, w, g = (t.to(DEV) for t in _gradient_inputs(shape, 73))
    code = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}[dtype]
    for query, call in ((kst.kst_backward_input_workspace_bytes, lambda ws: kst.kst_backward_input(g, w, N, P, ws=ws)),
                        (kst.kst_backward_weight_workspace_bytes, lambda ws: kst.kst_backward_weight(x, g, n, P, ws=ws))):
        need = query(B, Cin, Cout, N, n, P, code)
        full, accepted, refused = call(_scratch(need)), [], 0
        have = need
        while have > 64:                              # less and less of it
            have = have * 7 // 8 // 16 * 16
            try:
                accepted.append(call(_scratch(have)))
            except kst.KstError as e:
                assert e.status == 4                  # KST_ERR_WORKSPACE
                refused += 1
        other = [a for a in accepted if not torch.equal(a, full)]
        for a in other:                               # one alternative, the same every time
            assert torch.equal(a, other[0])
            assert float((a - full).abs().max()) <= 2 * TOL * float(full.abs().max())
        assert refused > 0
