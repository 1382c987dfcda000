"""The timed cases of this library: what a program that deploys a nested-integer model has it do, through the public
entry points (the ctypes binding and the network walker), from one small linear layer to a whole network.

    listed()             the cases, each a dict of plain values with a name
    draw(rng)            one more case from the same ranges
    prepare(case, seed)  inputs, weights and descriptors a program holds before the call
    run(state)           one pass; returns everything it computed
    work(case)           bytes and operations the pass cannot do without
    tolerance(case)      "exact": the path is integer sums and an fp32 epilogue with a fixed order of roundings

Kinds of case
    linear    one linear layer on int8 activations, fp32 out
    mlp       the two layers of a transformer MLP: D -> 4 D (int8 out, ReLU) -> D (fp32 out)
    words     a linear layer straight from pages in the 64-bit word layout (a model file used as it is)
    chain     convolution layers one after the other: dense, depthwise or grouped, bias, ReLU, int8 codes between them
    network   the ResNet-101 shaped network: one forward pass, or a switch (page-out, page-in beside a part-bit
              forward, full-bit forward)
    load      weights of a model on their way in: fp32 -> codes -> two packed pages, layer by layer
"""
from __future__ import annotations

import math

import torch

import paper_2506_17870_amd as nq
from paper_2506_17870_amd import network

STEP = 0.04          # quantisation step of int8 activations whose real values have unit variance
MAX_OPS = 2.2e11     # no drawn layer, MLP or chain is larger than this (multiply and add counted)


def _linear(M, K, N, n_bits=8, l_bits=2, full=True, signed=False):
    return dict(kind="linear", M=M, K=K, N=N, n_bits=n_bits, l_bits=l_bits, full=full, signed=signed)


def _mlp(M, D, n_bits=8, l_bits=3, full=True, signed=False):
    return dict(kind="mlp", M=M, D=D, n_bits=n_bits, l_bits=l_bits, full=full, signed=signed)


def _words(M, K, N, n_bits=8, l_bits=3, full=True, signed=False):
    return dict(kind="words", M=M, K=K, N=N, n_bits=n_bits, l_bits=l_bits, full=full, signed=signed)


def _chain(shape, B, H, n_bits=8, l_bits=2, full=True, signed=False, **sizes):
    return dict(kind="chain", shape=shape, B=B, H=H, n_bits=n_bits, l_bits=l_bits, full=full, signed=signed, **sizes)


def _network(B, switch, l_bits=2, full=True):
    return dict(kind="network", B=B, switch=switch, n_bits=8, l_bits=l_bits, full=full, signed=False)


def _load(layers, D, n_bits=8, l_bits=2, signed=False):
    return dict(kind="load", layers=layers, D=D, n_bits=n_bits, l_bits=l_bits, signed=signed)


def listed():
    return [
        # a single small layer called by itself: latency of one call
        dict(_linear(64, 512, 512), name="linear_64x512x512"),
        # a large layer with few rows, a decoding step or a small batch: the packed pages are the traffic
        dict(_linear(16, 8192, 8192), name="linear_16x8192x8192"),
        # the MLP of a ViT-B/16 layer for one image and for a batch of 64 (197 tokens each)
        dict(_mlp(197, 768), name="mlp_197x768"),
        dict(_mlp(12608, 768, full=False), name="mlp_12608x768_part"),
        # the same kind of layer from pages stored as the paper packs them, sizes that fit no tile
        dict(_words(197, 1000, 3000), name="words_197x1000x3000"),
        # a 3x3 convolution of a ResNet-18's first stage, fp32 out (the last layer handed to the caller)
        dict(_chain("conv", 32, 56, cin=64, cout=64, k=3, stride=1, int8=False), name="conv3x3_b32_56x56x64"),
        # a ResNet-101 stage-3 bottleneck block: 1x1, 3x3, 1x1 with residual
        dict(_chain("bottleneck", 64, 14, l_bits=4, width=256), name="bottleneck_b64_14x14x1024"),
        # depthwise + pointwise blocks of a MobileNet, strides included
        dict(_chain("separable", 32, 112, l_bits=3, cin=32, blocks=5), name="separable_b32_112x112x32"),
        # the grouped 3x3 layer of a ResNeXt block (32 groups of 8) between its 1x1 layers
        dict(_chain("grouped", 32, 56, l_bits=3, width=256, groups=32), name="grouped_b32_56x56x256_g32"),
        # a whole network for one image: a hundred small launches
        dict(_network(1, False), name="resnet101_b1"),
        # the whole network at a serving batch, switching from part-bit to full-bit
        dict(_network(128, True), name="resnet101_b128_switch"),
        # loading a model: quantise and pack the MLP weights of six transformer layers
        dict(_load(12, 768), name="load_12_layers_d768"),
    ]


# ---- more cases of the same ranges ---------------------------------------------------------------------------

NESTINGS = [(8, 1), (8, 2), (8, 3), (8, 4), (8, 5), (6, 1), (6, 2), (6, 3)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(rng, m, lo, hi):
    return max(lo, _log(rng, lo, hi) // m * m)


def draw(rng):
    kind = rng.choice(["linear", "linear", "mlp", "mlp", "words", "conv", "conv", "bottleneck", "separable", "grouped",
                       "network", "load"])
    n_bits, l_bits = rng.choice(NESTINGS)
    opt = dict(n_bits=n_bits, l_bits=l_bits, full=rng.random() < 0.6, signed=rng.random() < 0.15)
    while True:
        if kind == "linear":         # any number of rows and outputs; reductions in steps of 8
            c = _linear(_log(rng, 1, 8192), _mult(rng, 8, 64, 8192), _log(rng, 64, 8192), **opt)
        elif kind == "mlp":
            c = _mlp(_log(rng, 1, 12608), _mult(rng, 32, 192, 1536), **opt)
        elif kind == "words":        # any size at all
            c = _words(_log(rng, 1, 2048), _log(rng, 100, 8192), _log(rng, 100, 8192), **opt)
        elif kind == "conv":
            c = _chain("conv", _log(rng, 1, 64), _log(rng, 7, 112), cin=_mult(rng, 8, 16, 512), cout=_mult(rng, 8, 16, 512),
                       k=rng.choice([1, 3, 3, 3, 5]), stride=rng.choice([1, 1, 2]), int8=rng.random() < 0.7, **opt)
        elif kind == "bottleneck":
            c = _chain("bottleneck", _log(rng, 1, 128), rng.choice([7, 14, 20, 28, 33, 56]), width=_mult(rng, 16, 64, 512), **opt)
        elif kind == "separable":
            c = _chain("separable", _log(rng, 1, 32), rng.choice([14, 28, 50, 56, 112]), cin=_mult(rng, 8, 16, 128),
                       blocks=rng.randint(2, 5), **opt)
        elif kind == "grouped":
            groups = rng.choice([3, 8, 16, 32])
            c = _chain("grouped", _log(rng, 1, 32), _log(rng, 7, 56), width=groups * rng.choice([4, 8, 12, 16, 32]),
                       groups=groups, **opt)
        elif kind == "network":
            c = _network(_log(rng, 1, 100), rng.random() < 0.4, rng.choice([2, 3, 4]), rng.random() < 0.6)
        else:
            c = _load(rng.randint(2, 12), _mult(rng, 8, 128, 1024), n_bits, l_bits, opt["signed"])
        if kind == "network" or work(c)["flops"] <= MAX_OPS:
            return c


# ---- layers ---------------------------------------------------------------------------------------------------

def _conv_layers(c):
    """The layers of a chain: dicts of B, H, cin, cout, k, stride, pad, groups, relu, residual, int8."""
    B, H, out = c["B"], c["H"], []

    def add(cin, cout, k, stride=1, groups=1, relu=True, residual=False, int8=True):
        nonlocal H
        pad = k // 2
        out.append(dict(B=B, H=H, cin=cin, cout=cout, k=k, stride=stride, pad=pad, groups=groups, relu=relu,
                        residual=residual, int8=int8))
        H = (H + 2 * pad - k) // stride + 1

    if c["shape"] == "conv":
        add(c["cin"], c["cout"], c["k"], c["stride"], relu=c["int8"], int8=c["int8"])
    elif c["shape"] == "bottleneck":
        w = c["width"]
        add(4 * w, w, 1)
        add(w, w, 3)
        add(w, 4 * w, 1, residual=True)
    elif c["shape"] == "grouped":
        w = c["width"]
        add(w, w, 1)
        add(w, w, 3, groups=c["groups"])
        add(w, 2 * w, 1)
    else:                            # separable: depthwise 3x3, then 1x1; every second block halves the image
        cin = c["cin"]
        for i in range(c["blocks"]):
            cout = 2 * cin if i % 2 == 0 else cin
            add(cin, cin, 3, 2 if i % 2 == 1 else 1, groups=cin)
            add(cin, cout, 1)
            cin = cout
    return out


def _out_pixels(L):
    ho = (L["H"] + 2 * L["pad"] - L["k"]) // L["stride"] + 1
    return L["B"] * ho * ho


def _page_bytes(N, K, c, full=True):
    layout = nq.NQ_LAYOUT_PAPER_U64 if c["kind"] == "words" else nq.NQ_LAYOUT_DENSE
    low = c["l_bits"] + (1 if c["signed"] else 0)
    return nq.nq_packed_bytes(N, K, c["n_bits"] - c["l_bits"], layout) + (nq.nq_packed_bytes(N, K, low, layout) if full else 0)


def _network_work(c, full):
    """Of one forward pass: every activation tensor written once and read once per reader, pages once."""
    ops = network.resnet101_plan()
    hw, ch, B = {0: 224}, {0: 3}, c["B"]
    byts = flops = 0
    for op in ops:
        h, cin = hw[op["src"]], ch[op["src"]]
        byts += B * h * h * cin
        if op["op"] in ("conv", "maxpool"):
            ho = (h + 2 * op["pad"] - op["k"]) // op["stride"] + 1
        else:
            ho = 1
        cout = op.get("cout", cin)
        hw[op["dst"]], ch[op["dst"]] = ho, cout
        byts += B * ho * ho * cout * (4 if op["op"] == "fc" else (2 if op.get("residual") is not None else 1))
        if op["op"] in ("conv", "fc"):
            K = cin * op.get("k", 1) ** 2
            flops += 2 * B * ho * ho * cout * K
            byts += _page_bytes(cout, K, c, full) + 8 * cout
    return byts, flops


def _load_shapes(c):
    return [(4 * c["D"], c["D"]) if i % 2 == 0 else (c["D"], 4 * c["D"]) for i in range(c["layers"])]


def work(c):
    if c["kind"] in ("linear", "words"):
        M, K, N = c["M"], c["K"], c["N"]
        return dict(bytes=M * K + 4 * M * N + 4 * N + _page_bytes(N, K, c, c["full"]), flops=2 * M * N * K)
    if c["kind"] == "mlp":
        M, D = c["M"], c["D"]
        pages = _page_bytes(4 * D, D, c, c["full"]) + _page_bytes(D, 4 * D, c, c["full"])
        return dict(bytes=M * D + 2 * M * 4 * D + 4 * M * D + pages + 8 * 5 * D, flops=4 * M * D * 4 * D)
    if c["kind"] == "chain":
        byts = flops = 0
        for L in _conv_layers(c):
            K, m = L["k"] ** 2 * L["cin"] // L["groups"], _out_pixels(L)
            byts += L["B"] * L["H"] ** 2 * L["cin"] + m * L["cout"] * ((1 if L["int8"] else 4) + (1 if L["residual"] else 0))
            byts += _page_bytes(L["cout"], K, c, c["full"]) + 8 * L["cout"]
            flops += 2 * m * L["cout"] * K
        return dict(bytes=byts, flops=flops)
    if c["kind"] == "network":
        passes = [_network_work(c, f) for f in ((False, True) if c["switch"] else (c["full"],))]
        return dict(bytes=sum(p[0] for p in passes), flops=sum(p[1] for p in passes))
    byts = flops = 0
    for N, K in _load_shapes(c):
        byts += 4 * N * K + 4 * N + _page_bytes(N, K, c)
        flops += 2 * N * K
    return dict(bytes=byts, flops=flops)


def tolerance(c):
    return "exact"


# ---- inputs ---------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _cfg(c):
    return nq.make_cfg(c["n_bits"], c["l_bits"], nq.NQ_LOW_SIGNED_L1 if c["signed"] else nq.NQ_LOW_UNSIGNED_L,
                       nq.NQ_LAYOUT_PAPER_U64 if c["kind"] == "words" else nq.NQ_LAYOUT_DENSE)


def _weight(g, N, K, sigma, c):
    w = _randn(g, N, K) * sigma
    if c["kind"] != "words":
        return nq.NestedWeight.from_float(w, _cfg(c))
    codes = torch.empty((N, K), dtype=torch.int8, device="cuda")
    scale = torch.empty(N, dtype=torch.float32, device="cuda")
    nq.nq_quantize(w, N, K, c["n_bits"], codes, scale)
    return nq.NestedWeight.from_int8(codes, scale, _cfg(c))


def _codes(g, shape, c, relu):
    """int8 codes of N(0,1) activations (6-bit ones beside 6-bit weights), ReLU-clipped where a ReLU comes before."""
    q = 127 if c["n_bits"] == 8 else 31
    step = STEP * 127 / q
    v = torch.round(_randn(g, *shape) / step).clamp_(0 if relu else -q - 1, q).to(torch.int8)
    return v, step


def prepare(c, seed):
    g = _gen(seed)
    s = dict(case=c)
    if c["kind"] in ("linear", "words"):
        M, K, N = c["M"], c["K"], c["N"]
        s["w"] = _weight(g, N, K, 0.02, c)
        s["x"], step = _codes(g, (M, K), c, relu=False)
        s["epi"] = nq.make_epilogue(step)
        s["y"] = torch.empty((M, N), dtype=torch.float32, device="cuda")
    elif c["kind"] == "mlp":
        M, D = c["M"], c["D"]
        s["w1"], s["w2"] = _weight(g, 4 * D, D, (2 / D) ** 0.5, c), _weight(g, D, 4 * D, (0.5 / D) ** 0.5, c)
        s["b1"], s["b2"] = _randn(g, 4 * D) * 0.02, _randn(g, D) * 0.02
        s["x"], step = _codes(g, (M, D), c, relu=False)
        s["h"] = torch.empty((M, 4 * D), dtype=torch.int8, device="cuda")
        s["y"] = torch.empty((M, D), dtype=torch.float32, device="cuda")
        s["e1"] = nq.make_epilogue(step, s["b1"], relu=True, out_int8=True, inv_out_scale=1 / STEP)
        s["e2"] = nq.make_epilogue(STEP, s["b2"])
    elif c["kind"] == "chain":
        layers = _conv_layers(c)
        L = layers[0]
        s["x"], step = _codes(g, (L["B"], L["H"], L["H"], L["cin"]), c, relu=True)
        s["steps"] = []
        src = s["x"]
        for L in layers:
            K = L["k"] ** 2 * L["cin"] // L["groups"]
            w = _weight(g, L["cout"], K, (2 / K) ** 0.5, c)
            bias = _randn(g, L["cout"]) * 0.02
            ho = (L["H"] + 2 * L["pad"] - L["k"]) // L["stride"] + 1
            y = torch.empty((L["B"], ho, ho, L["cout"]), dtype=torch.int8 if L["int8"] else torch.float32, device="cuda")
            res = s["x"] if L["residual"] else None
            epi = nq.make_epilogue(step, bias, res, STEP if L["residual"] else 0.0, relu=L["relu"], out_int8=L["int8"],
                                   inv_out_scale=1 / STEP)
            shape = nq.nq_conv_shape(L["B"], L["H"], L["H"], L["cin"], L["cout"], L["k"], L["k"], L["stride"], L["pad"])
            s["steps"].append((L["groups"], src, shape, w, epi, y, bias))
            src, step = y, STEP
    elif c["kind"] == "network":
        ops = network.resnet101_plan()
        weights = []
        for op in ops:
            if op["op"] not in ("conv", "fc"):
                weights.append(None)
                continue
            K = op.get("k", 1) ** 2 * op["cin"]
            weights.append(((_randn(g, op["cout"], K) * (2 / K) ** 0.5).cpu().numpy(),
                            (_randn(g, op["cout"]) * 0.02).cpu().numpy()))
        s["net"] = network.NestedCNN(ops, weights, c["n_bits"], c["l_bits"])
        s["x"], s["step"] = network.quantize_tensor(_randn(g, c["B"], 224, 224, 3))
        s["net"].calibrate(s["x"], s["step"])
        s["copy"] = torch.cuda.Stream()
    else:
        s["jobs"] = []
        for N, K in _load_shapes(c):
            high = torch.empty(nq.nq_packed_bytes(N, K, c["n_bits"] - c["l_bits"]), dtype=torch.uint8, device="cuda")
            low = torch.empty(nq.nq_packed_bytes(N, K, c["l_bits"] + (1 if c["signed"] else 0)), dtype=torch.uint8, device="cuda")
            scale = torch.empty(N, dtype=torch.float32, device="cuda")
            s["jobs"].append((_randn(g, N, K) * (2 / K) ** 0.5, N, K, scale, high, low))
        s["cfg"] = _cfg(c)
    return s


# ---- one pass ---------------------------------------------------------------------------------------------------

def run(s):
    c = s["case"]
    if c["kind"] in ("linear", "words"):
        (nq.nq_gemm_full if c["full"] else nq.nq_gemm_part)(s["x"], c["M"], s["w"].desc, s["epi"], s["y"])
        return s["y"]
    if c["kind"] == "mlp":
        gemm = nq.nq_gemm_full if c["full"] else nq.nq_gemm_part
        gemm(s["x"], c["M"], s["w1"].desc, s["e1"], s["h"])
        gemm(s["h"], c["M"], s["w2"].desc, s["e2"], s["y"])
        return s["h"], s["y"]
    if c["kind"] == "chain":
        conv, gconv = (nq.nq_conv_full, nq.nq_gconv_full) if c["full"] else (nq.nq_conv_part, nq.nq_gconv_part)
        for groups, x, shape, w, epi, y, _ in s["steps"]:
            if groups == 1:
                conv(x, shape, w.desc, epi, y)
            else:
                gconv(x, shape, groups, w.desc, epi, y)
        return tuple(step[5] for step in s["steps"])
    if c["kind"] == "network":
        net = s["net"]
        if not c["switch"]:
            return net.forward(s["x"], s["step"], c["full"])
        net.page_out_low()                                   # the model serves part-bit ...
        net.page_in_low(s["copy"])                           # ... while its lower-bit pages come back
        part = net.forward(s["x"], s["step"], False).clone()
        return part, net.forward(s["x"], s["step"], True)    # waits for the pages on the device
    for w, N, K, scale, high, low in s["jobs"]:
        nq.nq_quantize_decompose_pack(w, N, K, s["cfg"], scale, high, low)
    return [(scale, high, low) for _, _, _, scale, high, low in s["jobs"]]
