"""The kernels that split fp32 operands for the bf16 matrix cores, as far as they show without a GPU: what their three
parts keep of a value, which layers they take, and their workspaces against what they lay out in them."""
import pytest
import torch

from paper_2209_03704_amd import binding as kst

F32, BF16, F16 = kst.KST_F32, kst.KST_BF16, kst.KST_F16


def _up(v, to):
    return (v + to - 1) // to * to


def split_din_weight_bytes(Cin, Cout, n, parts):
    """[block of 32 input channels][chunk of 16 output channels][tap][part][64 lanes][8 values of 2 bytes]"""
    return _up(_up(Cin, 32) // 32 * (_up(Cout, 16) // 16) * n * n * parts * 1024, 256)


def slot_count(grid, passes):
    """Partial tiles of `passes` tiles shared by `grid` workgroups: one per workgroup and tile, or two per workgroup."""
    return 0 if passes == 0 else grid + passes - 1 if passes < grid else 2 * grid


def split_din_slot_bytes(B, Cin, Cout, N, n):
    """Partial tiles of 128 positions and 128 or 256 input channels."""
    tiles_m, chunks = -(-B * N * N // 128), -(-Cout // 16)
    rb = 2 if n < 5 and Cin > 128 and tiles_m * -(-Cin // 256) * chunks >= 4 * 256 else 1
    tiles = tiles_m * -(-Cin // (128 * rb))
    return slot_count(min(256, tiles * chunks), tiles % 256) * rb * 256 * 64 * 4


def split_forward_bytes(B, Cin, Cout, N, n, P):
    """Split weights [row parity][block of 32 output channels][chunk][tap][part][64 lanes][8 values], then partial tiles
    of 128 positions x 128 output channels (256 x 64 up to 64 channels) of one row parity."""
    E = -(-(2 * (N + 2 * ((P + 1) // 2)) - n) // 2)
    wide = Cout > 64
    tiles = -(-B * E * E // (128 if wide else 256)) * -(-Cout // (128 if wide else 64))
    chunks = -(-Cin // 16)
    per_round = 256 if n % 2 == 0 else 512                  # (odd kernels: the two parities cost differently, so pairs)
    passes = 2 * tiles % per_round
    weights = _up(-(-Cout // 32) * chunks * n * n * 3 * 1024, 256)
    return weights + slot_count(min(256, 2 * tiles * chunks), passes) * 256 * 128 * 4


def split_dw_bytes(B, Cin, Cout, N, n, P, parts):
    """Operands [block of 32 channels][position][16 items][part][64 lanes][8 values] of the input (`parts`) and of g
    (three), then partial sums [split][tap][co][ci]."""
    M, groups = 2 * N + 2 * P - n, -(-B // 16)
    steps, tiles = N * N * groups, -(-Cout // 128) * -(-Cin // 128) * ((n * n + 1) // 2)
    splits = max(1, min(256 // tiles if tiles < 256 else 1, steps // 16))
    per = (-(-steps // splits) + 1) // 2 * 2
    splits = -(-steps // per)
    return (-(-Cin // 32) * N * N * groups * parts * 1024 + -(-Cout // 32) * M * M * groups * 3 * 1024 +
            _up(splits * n * n * Cout * Cin * 4, 256))


def split_din_query(B, Cin, Cout, N, n, P, dtype):
    """16-bit weights: with their widened copy (bfloat16 does without; the query gives one size)."""
    widened = _up(Cin * Cout * n * n * 4, 256) if dtype != F32 else 0
    return widened + split_din_weight_bytes(Cin, Cout, n, 3) + split_din_slot_bytes(B, Cin, Cout, N, n)


def split_dw_query(B, Cin, Cout, N, n, P, dtype):
    """16-bit input: with its widened copy, which only the kernels that multiply in fp32 read."""
    return split_dw_bytes(B, Cin, Cout, N, n, P, 3) + (_up(B * Cin * N * N * 4, 256) if dtype != F32 else 0)


# ---- variants of the kernels: which one a layer runs ----------------------------------------------------------------

def forward_variant(B, Cin, Cout, N, n, P):
    """(kernel edge, 128 or 64 output channels per tile, staged positions per lane), None for a map these do not take."""
    Nq = N + 2 * ((P + 1) // 2)
    E = -(-(2 * Nq - n) // 2)
    steps = ((128 if Cout > 64 else 256) - 2) // E + 1
    staged = (steps + (steps + E - 1) // E * (Nq - E) + n // 2 + 1) * Nq
    return (n, 128 if Cout > 64 else 64, 3 if staged <= 384 else 5) if staged <= 640 else None


def input_gradient_variant(B, Cin, Cout, N, n, P, dtype):
    """(kernel edge, 256 or 128 input channels per tile, parts of the weights, staged cells per lane), or None."""
    tiles_m, chunks = -(-B * N * N // 128), -(-Cout // 16)
    two = n < 5 and Cin > 128 and tiles_m * -(-Cin // 256) * chunks >= 4 * 256
    rows = 128 // N
    whole = rows * N == 128 and (rows % N == 0 or N % rows == 0)
    steps = rows - 1 if whole else 126 // N + 1
    items = (rows - 1) // N if whole else (steps + N - 1) // N
    staged = (2 * steps + items * (n - 2) + n) * 2 * ((2 * N + n - 1) // 2)
    return (n, 256 if two else 128, 1 if dtype == "bf16" else 3, 5 if staged <= 640 else 7) if staged <= 832 else None


# Weights whose three parts pass the 2 GB a launch can address while bfloat16's one part does not: the size has to be
# that of the type that is launched, from the first byte the launch writes to its last.
@pytest.mark.parametrize("B,Cin,Cout,N,n", [(1, 7000, 7000, 8, 4), (1, 10000, 10000, 8, 3), (1, 6000, 6000, 8, 5)])
def test_bf16_input_gradient_workspace_holds_large_weights(B, Cin, Cout, N, n):
    assert split_din_weight_bytes(Cin, Cout, n, 1) < 2 ** 31 <= split_din_weight_bytes(Cin, Cout, n, 3)
    laid_out = split_din_weight_bytes(Cin, Cout, n, 1) + split_din_slot_bytes(B, Cin, Cout, N, n)
    assert kst.kst_backward_input_workspace_bytes(B, Cin, Cout, N, n, 0, BF16) == laid_out
    # a byte less is refused before anything is launched (pointers are never followed)
    assert kst.lib().kst_backward_input(16, 16, 16, 16, laid_out - 1, B, Cin, Cout, N, n, 0, BF16, None) == 4
    # three parts: not these kernels (half precision is widened to fp32 first, fp32 weights are their own)
    for dt in (F32, F16):
        assert kst.kst_backward_input_workspace_bytes(B, Cin, Cout, N, n, 0, dt) != (
            split_din_weight_bytes(Cin, Cout, n, 3) + split_din_slot_bytes(B, Cin, Cout, N, n))


@pytest.mark.parametrize("B,Cin,Cout,N,n", [(64, 512, 256, 8, 4), (160, 250, 130, 10, 3), (256, 128, 96, 8, 5)])
def test_input_gradient_workspace_is_the_layout(B, Cin, Cout, N, n):
    slots = split_din_slot_bytes(B, Cin, Cout, N, n)
    widened = _up(Cin * Cout * n * n * 4, 256)
    of = {dt: kst.kst_backward_input_workspace_bytes(B, Cin, Cout, N, n, 0, dt) for dt in (F32, BF16, F16)}
    assert of[F32] == split_din_weight_bytes(Cin, Cout, n, 3) + slots
    assert of[F16] == widened + of[F32]
    assert of[BF16] == of[F16] > split_din_weight_bytes(Cin, Cout, n, 1) + slots      # one size for 16-bit types


# Shared passes only; whole rounds and shared passes; more shared passes than workgroups; tiles of 64 channels.
@pytest.mark.parametrize("B,Cin,Cout,N,n,P", [(64, 512, 256, 8, 4, 2), (128, 512, 256, 16, 4, 0), (64, 1024, 512, 8, 5, 0),
                                              (23, 515, 264, 13, 3, 2), (70, 33, 40, 33, 5, 1)])
def test_forward_workspace_is_the_layout(B, Cin, Cout, N, n, P):
    assert kst.kst_workspace_bytes_padded(B, Cin, Cout, N, n, P, F32) == split_forward_bytes(B, Cin, Cout, N, n, P)
    if P == 0:
        assert kst.kst_workspace_bytes(B, Cin, Cout, N, n, F32) == split_forward_bytes(B, Cin, Cout, N, n, P)


def test_partial_tiles_are_numbered_along_the_list():
    """128 shared passes of 256 workgroups: 383 slots of 128 KB and 12.6 MB of split weights, where two slots per
    workgroup made 79.7 MB, more than the library's fixed workspace holds."""
    need = kst.kst_workspace_bytes_padded(64, 512, 256, 8, 4, 2, F32)
    assert need == 383 * 131072 + 12582912 < kst.KST_STATIC_SCRATCH_BYTES


# Which layers run on the split kernels: either side of each rule's line, told by the workspace.
@pytest.mark.parametrize("shape,split", [
    ((36, 896, 128, 4, 5, 1), False),     # ten passes of 56 chunks: mostly partial tiles
    ((6, 128, 128, 48, 3, 1), False),     # short passes
    ((10, 96, 192, 64, 3, 2), False),     # fewer than eight chunks, whatever the size
    ((10, 98, 192, 64, 3, 2), True),      # ... where the pipelined fp32 kernel does not apply (no groups of four)
    ((16, 512, 256, 8, 4, 2), True),      # 2.1 G products, whole chunks
    ((8, 512, 256, 8, 4, 2), False),      # 1.1 G
    ((3, 1024, 512, 10, 5, 2), True),     # 3.9 G, shared by few passes
    ((40, 128, 256, 16, 4, 2), True),     # from 4 G always
])
def test_forward_route(shape, split):
    assert (kst.kst_workspace_bytes_padded(*shape, F32) == split_forward_bytes(*shape)) == split


@pytest.mark.parametrize("shape,split", [
    ((13, 768, 384, 6, 4, 2), False),     # 2.2 G, the pipelined fp32 kernel at its best
    ((13, 768, 383, 6, 4, 2), True),      # ... which wants whole groups of four channels
    ((16, 768, 384, 6, 4, 2), True),      # 2.7 G
    ((20, 256, 256, 8, 5, 0), False),     # 2.1 G
    ((21, 256, 256, 8, 5, 0), True),      # 2.2 G
])
def test_input_gradient_route(shape, split):
    assert (kst.kst_backward_input_workspace_bytes(*shape, F32) == split_din_query(*shape, F32)) == split


def test_input_gradient_route_of_one_part():
    """bfloat16 weights from 2.2 G whatever the other kernel is (both queries are half precision's where that one also
    runs split, the launch's own where it does not)."""
    B, Cin, Cout, N, n, P = shape = (13, 768, 384, 6, 4, 2)
    assert kst.kst_backward_input_workspace_bytes(*shape, BF16) == (
        split_din_weight_bytes(Cin, Cout, n, 1) + split_din_slot_bytes(B, Cin, Cout, N, n))
    assert kst.kst_backward_input_workspace_bytes(*shape, F16) != split_din_query(*shape, F16)


@pytest.mark.parametrize("shape,dtype,split", [
    ((68, 128, 128, 24, 3, 3), F32, False),    # 9 products per value of g and input channel, one tile of those
    ((68, 128, 128, 24, 3, 3), BF16, True),    # (bfloat16 input: half the multiplies)
    ((68, 130, 128, 25, 3, 3), F32, False),    # half of the second tile of input channels would be padding
    ((68, 256, 128, 24, 3, 3), F32, True),
    ((68, 128, 128, 23, 3, 3), F32, True),     # columns no whole groups of four
    ((64, 512, 256, 8, 4, 2), F32, True),
    ((16, 512, 256, 8, 4, 2), F32, False),     # 2.1 G products
])
def test_kernel_gradient_route(shape, dtype, split):
    assert (kst.kst_backward_weight_workspace_bytes(*shape, dtype) == split_dw_query(*shape, dtype)) == split


def test_three_parts_of_every_fp32_value():
    """Every mantissa at exponents from the subnormal ones up: the parts of the value times 2^24 add up to it, are normal
    bfloat16 numbers (or zero), and are as small as the error bound of a product takes them to be."""
    mantissas = torch.arange(1 << 23, dtype=torch.int32)
    for exponent in (0, 1, 17, 127, 228):
        x = ((exponent << 23) | mantissas).view(torch.float32) * 2.0 ** 24
        p0 = x.bfloat16().float()
        p1 = (x - p0).bfloat16().float()
        p2 = x - p0 - p1
        assert torch.equal(p2.bfloat16().float(), p2)
        assert (p1.abs() <= 2.0 ** -8 * x).all() and (p2.abs() <= 2.0 ** -17 * x).all()
        for part in (p0, p1, p2):
            assert part[part != 0].abs().min() >= 2.0 ** -126
        # what a product of x with itself leaves out: x1 x2 twice and x2 x2
        left = (2 * p1.double() * p2.double() + p2.double() ** 2).abs()
        assert (left <= 2.0 ** -24 * x.double() ** 2).all()


def test_gpu_shapes_run_every_variant():
    """The layers the GPU tests run, against every variant any map edge and channel count leads to."""
    import test_gpu_split as gpu
    edges, pads = range(4, 132), range(4)
    forward = {forward_variant(1, 32, Cout, N, n, P) for n in (3, 4, 5) for N in edges for P in pads for Cout in (48, 130)}
    assert {forward_variant(*s) for s in gpu.FORWARD} == forward - {None}
    gradient = {input_gradient_variant(B, Cin, 256, N, n, 0, dt) for n in (3, 4, 5) for N in edges
                for B, Cin in ((64, 100), (640, 300)) for dt in ("f32", "bf16")}
    assert {input_gradient_variant(*s) for s in gpu.INPUT_GRADIENT} == gradient - {None}
    assert {(s[4], s[6]) for s in gpu.KERNEL_GRADIENT} == {(n, dt) for n in (3, 4, 5) for dt in ("f32", "bf16", "f16")}


def test_maps_the_input_gradient_takes():
    """Its stage of 832 cells holds the rows of g that 128 positions touch on these maps only."""
    takes = lambda n: [N for N in range(4, 132) if input_gradient_variant(1, 64, 64, N, n, 0, "f32")]
    assert takes(3) == [*range(4, 29), 32, 33, 64, 128]
    assert takes(4) == [*range(4, 18), 19, 22, 32, 64]
    assert takes(5) == [8, 16, 32]
    for n in (3, 4, 5):
        for N in range(4, 70):
            B = max(1, -(-int(4e9) // (N * N * n * n * 128 * 66)))
            if (2 * N - n) > 0 and B * 66 * (2 * N) ** 2 * 4 < 2 ** 31:
                need = kst.kst_backward_input_workspace_bytes(B, 100, 66, N, n, 0, F32)
                assert (need == split_din_query(B, 100, 66, N, n, 0, F32)) == (N in takes(n)), (n, N)
