"""Timed cases of the library's public entry points: what they are, how their inputs are made,
one pass of each, the work a pass cannot do without, and its result in 64 bits.

A case is a dict of plain values:
    op      what one pass calls
              "whole"      kst_forward / kst_forward_padded from un-segregated weights
              "forward"    kst_forward_seg_epilogue (kst_forward_seg_padded where the layer has
                           neither bias nor activation) on weights segregated beforehand
              "generator"  a generator's transpose-convolution layers one after the other, each with
                           its bias and activation; the outputs of all layers are returned
              "gradients"  kst_backward_input and kst_backward_weight
              "train"      the forward pass and both gradients of one layer
    B, Cin, Cout, N, n, P, dtype       the layer as in include/kst.h
    bias, act                          its epilogue (op "forward")
    dist    distribution of the input: "uniform" [-1, 1], "normal", "relu_normal"
    layers  op "generator": "N:Cin:Cout" per layer, kernel edge n and padding factor P for all

Buffers a program keeps between calls (outputs, workspaces, segregated weights) are made in
prepare().
"""
from __future__ import annotations

import math

import torch

from paper_2209_03704_amd import binding as kst

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_CODES = {"f32": kst.KST_F32, "bf16": kst.KST_BF16, "f16": kst.KST_F16}
_ACTS = {"none": kst.KST_ACT_NONE, "relu": kst.KST_ACT_RELU, "tanh": kst.KST_ACT_TANH}


def _case(name, op, B, Cin, Cout, N, n, P=0, dtype="f32", dist="relu_normal", bias=False, act="none", layers=""):
    return {"name": name, "op": op, "B": B, "Cin": Cin, "Cout": Cout, "N": N, "n": n, "P": P, "dtype": dtype,
            "dist": dist, "bias": bias, "act": act, "layers": layers}


_DCGAN = "4:1024:512 8:512:256 16:256:128 32:128:3"


def listed():
    return [
        # One small image map, weights as they come: the smallest call, all launch latency.
        _case("whole_tiny_map", "whole", 1, 1, 1, 32, 3, dist="uniform"),
        # Up-scaling a batch of large single-channel maps: the memory-bound headline layer.
        _case("maps_1ch_512", "forward", 64, 1, 1, 512, 5, dist="normal"),
        # A data set's colour images (224 x 224 x 3) up-scaled with the largest kernel of Table 1.
        _case("images_224_n5", "forward", 256, 3, 1, 224, 5, P=2, dist="uniform"),
        # Learning such an image layer's kernel, and the gradient handed to the layer before it.
        _case("images_224_n3_gradients", "gradients", 128, 3, 1, 224, 3, P=2, dist="uniform"),
        # A generator's wide middle layer at a large batch, unpadded.
        _case("gan_n4_f32", "forward", 128, 512, 256, 16, 4),
        # A generator's first layer: deep channels, small odd map, bias and ReLU as it is used.
        _case("deep_n5_f32", "forward", 64, 1024, 512, 8, 5, bias=True, act="relu"),
        # A generator's late layer in bfloat16: wide maps, the output is most of the traffic.
        _case("late_n3_bf16", "forward", 32, 256, 128, 64, 3, dtype="bf16"),
        # Sampling: one latent through all transpose-convolution layers of the DCGAN generator.
        _case("dcgan_one_sample", "generator", 1, 1024, 3, 4, 4, P=2, layers=_DCGAN),
        # Training a DCGAN layer in fp32: forward, input gradient, kernel gradient.
        _case("dcgan_l3_train", "train", 64, 512, 256, 8, 4, P=2),
        # ... the generator's output layer, few output channels.
        _case("dcgan_l5_train", "train", 64, 128, 3, 32, 4, P=2),
        # ... and a layer with bfloat16 operands.
        _case("dcgan_l4_train_bf16", "train", 64, 256, 128, 16, 4, P=2, dtype="bf16"),
        # Ragged channel counts, odd map, odd padding factor, half precision, weights as they come.
        _case("whole_ragged_f16", "whole", 24, 100, 52, 19, 3, P=1, dtype="f16"),
    ]


def draw(rng):
    """One more case of the same kinds.  At most 4 G multiply-adds and about 48 M elements a pass."""
    def logi(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["image", "image_gradients", "map", "channels", "channels", "train", "train", "one_sample"])
    n, P = rng.choice([3, 4, 5]), rng.choice([0, 1, 2, 2, 3])
    dtype, dist, bias, act, op = "f32", "relu_normal", False, "none", "forward"
    if kind == "map":
        Cin, Cout, N, dist = 1, 1, logi(32, 512), "normal"
    elif kind in ("image", "image_gradients"):
        Cin, Cout, N, dist = 3, 1, logi(64, 256), "uniform"
        op = "gradients" if kind == "image_gradients" else "forward"
    elif kind == "one_sample":
        N = rng.choice([4, 8, 16, 32])
        Cin, Cout = logi(64, 4096 // N), logi(3, 2048 // N)
        bias, act = True, rng.choice(["relu", "tanh"])
    else:
        N = logi(4, 64)
        Cin = rng.choice([logi(16, 1024), 4 * logi(8, 256), 32 * logi(1, 16)])
        Cout = rng.choice([logi(16, 512), 4 * logi(4, 128), 32 * logi(1, 16), 3])
        dtype = rng.choice(["f32", "f32", "bf16", "f16"])
        op = "train" if kind == "train" else rng.choice(["forward", "forward", "whole"])
        if op == "forward" and rng.random() < 0.5:
            bias, act = True, rng.choice(["relu", "tanh", "none"])
    passes = {"train": 3, "gradients": 2}.get(op, 1)
    case = _case("", op, 1, Cin, Cout, N, n, P, dtype, dist, bias, act)
    while _layer_macs(case) * passes > 4.0e9:
        case["N"] = N = N * 3 // 4
    if kind != "one_sample":
        one = _layer_macs(case) * passes
        elems = Cin * N * N + Cout * _edge(N, n, P) ** 2
        most = min(4.0e9 / one, (48.0e6 - Cin * Cout * n * n) / elems, 256)
        case["B"] = max(1, min(logi(1, 256), int(most)))
    return {k: v for k, v in case.items() if k != "name"}


def _edge(N, n, P):
    return 2 * N + 2 * P - n


def _layer_macs(c):
    """Products with an original input pixel whose output lies inside the map, all channels."""
    M = _edge(c["N"], c["n"], c["P"])
    hits = sum(max(0, min(c["N"] - 1, (M - 1 + u - c["P"]) // 2) - max(0, -((c["P"] - u) // 2)) + 1)
               for u in range(c["n"]))
    return hits * hits * c["B"] * c["Cin"] * c["Cout"]


def _generator_layers(c):
    out = []
    for i, part in enumerate(c["layers"].split()):
        N, Cin, Cout = (int(v) for v in part.split(":"))
        last = i == len(c["layers"].split()) - 1
        out.append(dict(c, op="forward", N=N, Cin=Cin, Cout=Cout, bias=True, act="tanh" if last else "relu"))
    return out


def work(case):
    if case["op"] == "generator":
        parts = [work(c) for c in _generator_layers(case)]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    c = case
    size = 4 if c["dtype"] == "f32" else 2
    x = c["B"] * c["Cin"] * c["N"] ** 2
    w = c["Cout"] * c["Cin"] * c["n"] ** 2
    o = c["B"] * c["Cout"] * _edge(c["N"], c["n"], c["P"]) ** 2
    forward = (x + w) * size + o * 4 + (c["Cout"] * 4 if c["bias"] else 0)
    grads = (w + x) * size + o * 4 + (x + w) * 4
    macs = _layer_macs(c)
    return {"whole": {"bytes": forward, "flops": 2 * macs},
            "forward": {"bytes": forward, "flops": 2 * macs},
            "gradients": {"bytes": grads, "flops": 4 * macs},
            # in, w and g are read once, out and both gradients written once
            "train": {"bytes": grads + o * 4, "flops": 6 * macs}}[c["op"]]


def _inputs(case, seed):
    """(x, w, bias, g) of one layer on the GPU, from the seed alone."""
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = _DTYPES[c["dtype"]]
    shape = (c["B"], c["Cin"], c["N"], c["N"])
    if c["dist"] == "uniform":
        x = torch.rand(shape, generator=gen, device="cuda").mul_(2.0).sub_(1.0)
    else:
        x = torch.randn(shape, generator=gen, device="cuda")
        if c["dist"] == "relu_normal":
            x.clamp_(min=0.0)
    w = torch.randn((c["Cout"], c["Cin"], c["n"], c["n"]), generator=gen, device="cuda").mul_(0.02)
    bias = torch.randn(c["Cout"], generator=gen, device="cuda").mul_(0.1) if c["bias"] else None
    g = None
    if c["op"] in ("train", "gradients"):
        M = _edge(c["N"], c["n"], c["P"])
        g = torch.randn((c["B"], c["Cout"], M, M), generator=gen, device="cuda").mul_(0.05)
    return x.to(dt), w.to(dt), bias, g


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None


def prepare(case, seed):
    if case["op"] == "generator":
        layers = _generator_layers(case)
        parts = [prepare(c, seed * 16 + i) for i, c in enumerate(layers)]
        return {"case": case, "parts": parts, "x": parts[0]["x"]}
    c = case
    x, w, bias, g = _inputs(c, seed)
    dims = (c["B"], c["Cin"], c["Cout"], c["N"], c["n"], c["P"], _CODES[c["dtype"]])
    M = _edge(c["N"], c["n"], c["P"])
    st = {"case": c, "x": x, "w": w, "bias": bias, "g": g}
    if c["op"] != "gradients":
        st["out"] = torch.empty((c["B"], c["Cout"], M, M), device="cuda")
    if c["op"] in ("forward", "train"):
        st["w_seg"] = kst.kst_segregate_weights(w)
        st["ws"] = _workspace(kst.kst_workspace_bytes_padded(*dims))
    if c["op"] in ("train", "gradients"):
        st["din"] = torch.empty(x.shape, device="cuda")
        st["dw"] = torch.empty(w.shape, device="cuda")
        st["ws_in"] = _workspace(kst.kst_backward_input_workspace_bytes(*dims))
        st["ws_w"] = _workspace(kst.kst_backward_weight_workspace_bytes(*dims))
    return st


def _forward(st, x):
    c = st["case"]
    if c["bias"] or c["act"] != "none":
        return kst.kst_forward_seg_epilogue(x, st["w_seg"], c["Cout"], c["n"], bias=st["bias"], act=_ACTS[c["act"]],
                                            P=c["P"], out=st["out"], ws=st["ws"])
    return kst.kst_forward_seg_padded(x, st["w_seg"], c["Cout"], c["n"], c["P"], out=st["out"], ws=st["ws"])


def run(state):
    st, c = state, state["case"]
    if c["op"] == "generator":
        outs, x = [], st["x"]
        for part in st["parts"]:
            x = _forward(part, x)
            outs.append(x)
        return outs
    if c["op"] == "whole":
        if c["P"] == 0:
            return kst.kst_forward(st["x"], st["w"], out=st["out"])
        return kst.kst_forward_padded(st["x"], st["w"], c["P"], out=st["out"])
    if c["op"] == "forward":
        return _forward(st, st["x"])
    outs = [_forward(st, st["x"])] if c["op"] == "train" else []
    outs.append(kst.kst_backward_input(st["g"], st["w"], c["N"], c["P"], din=st["din"], ws=st["ws_in"]))
    outs.append(kst.kst_backward_weight(st["x"], st["g"], c["n"], c["P"], dw=st["dw"], ws=st["ws_w"]))
    return outs


def tolerance(case):
    # Every operand type: products of 16-bit operands are exact in fp32 and all sums are fp32, so what
    # differs between correct implementations is the order of the sums.
    return {"rel": 4e-6, "max": 4e-5}


# ---- the same results in 64 bits, by the definition's index relation -------------------------

def _tap_range(c, M, u):
    """Input rows a with 0 <= 2a + P - u < M: (first, last + 1, first output row)."""
    lo = max(0, -((c["P"] - u) // 2))
    hi = min(c["N"] - 1, (M - 1 + u - c["P"]) // 2) + 1
    return lo, hi, 2 * lo + c["P"] - u


def _exact_forward(c, x, w, bias):
    B, Cin, Cout, N, n = c["B"], c["Cin"], c["Cout"], c["N"], c["n"]
    M = _edge(N, n, c["P"])
    out = torch.zeros((Cout, B, M, M), dtype=torch.float64, device=x.device)
    xt = x.double().transpose(0, 1).contiguous().view(Cin, B * N * N)
    w = w.double()
    for u in range(n):
        a0, a1, y0 = _tap_range(c, M, u)
        for v in range(n):
            c0, c1, x0 = _tap_range(c, M, v)
            if a0 >= a1 or c0 >= c1:
                continue
            t = (w[:, :, u, v].contiguous() @ xt).view(Cout, B, N, N)
            out[:, :, y0:y0 + 2 * (a1 - a0) - 1:2, x0:x0 + 2 * (c1 - c0) - 1:2] += t[:, :, a0:a1, c0:c1]
    out = out.transpose(0, 1).contiguous()
    if bias is not None:
        out += bias.double().view(1, Cout, 1, 1)
    if c["act"] == "relu":
        out.clamp_(min=0.0)
    elif c["act"] == "tanh":
        out.tanh_()
    return out


def _exact_gradients(c, x, w, g):
    B, Cin, Cout, N, n = c["B"], c["Cin"], c["Cout"], c["N"], c["n"]
    M = _edge(N, n, c["P"])
    xt = x.double().transpose(0, 1).contiguous().view(Cin, B * N * N)
    gt = g.double().transpose(0, 1).contiguous()
    w = w.double()
    din = torch.zeros((Cin, B * N * N), dtype=torch.float64, device=x.device)
    dw = torch.zeros((Cout, Cin, n, n), dtype=torch.float64, device=x.device)
    for u in range(n):
        a0, a1, y0 = _tap_range(c, M, u)
        for v in range(n):
            c0, c1, x0 = _tap_range(c, M, v)
            if a0 >= a1 or c0 >= c1:
                continue
            t = torch.zeros((Cout, B, N, N), dtype=torch.float64, device=x.device)
            t[:, :, a0:a1, c0:c1] = gt[:, :, y0:y0 + 2 * (a1 - a0) - 1:2, x0:x0 + 2 * (c1 - c0) - 1:2]
            t = t.view(Cout, B * N * N)
            din += w[:, :, u, v].t().contiguous() @ t
            dw[:, :, u, v] = t @ xt.t().contiguous()
    return din.view(Cin, B, N, N).transpose(0, 1).contiguous(), dw


def exact(case, seed):
    if case["op"] == "generator":
        outs, x = [], None
        for i, c in enumerate(_generator_layers(case)):
            first, w, bias, _ = _inputs(c, seed * 16 + i)
            x = first if x is None else x
            x = _exact_forward(c, x, w, bias)
            outs.append(x)
        return outs
    x, w, bias, g = _inputs(case, seed)
    outs = []
    if case["op"] != "gradients":
        outs.append(_exact_forward(case, x, w, bias))
    if case["op"] in ("train", "gradients"):
        outs.extend(_exact_gradients(case, x, w, g))
    return outs if case["op"] in ("train", "gradients") else outs[0]
