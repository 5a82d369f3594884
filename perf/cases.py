"""The work that programs have this library do, as cases that can be measured.

A case is a dict of plain values with an "op":
  fc         one binary fully connected layer on fp32 activations (binary_fc)
  fc_pair    two of them in a row, the second on the fp32 result of the first
  fc_bits    the same pair handing packed sign bits on (binarize_pack, binary_fc_packed twice)
  conv       one binary convolution on an fp32 NCHW image (binary_conv2d)
  conv_bits  three convolutions that hand packed images on (pack_nchw, binary_conv2d_bits twice,
             binary_conv2d_packed), thresholds as a folded BatchNorm leaves them
  quant      k-bit activations against 1-bit or k-bit weights (quant_gemm)
  gemm       the xnor product of two packed matrices, in rows of 64-bit or 32-bit words
  convert    fp32 weights to packed bits and their scale (the converter's step of a model)
Layers have their weights packed and scaled in prepare(): a program does that once, offline.
"""
import math

import torch

from paper_1705_09864_amd import binding as B


def listed():
    return [
        # the smallest layer a program calls: a microsecond of work, so latency is all there is
        {"name": "fc_small", "op": "fc", "batch": 64, "fin": 512, "fout": 256, "out": "i32"},
        # one request through an AlexNet-sized classifier layer: a matrix-vector product
        {"name": "fc_one_request", "op": "fc", "batch": 1, "fin": 9216, "fout": 4096, "out": "f32"},
        # row lengths that are no whole number of words, with an odd number of them
        {"name": "fc_ragged", "op": "fc", "batch": 100, "fin": 2100, "fout": 1000, "out": "f32"},
        # the AlexNet classifier at batch 256, in a loop that keeps its buffers
        {"name": "fc_pair", "op": "fc_pair", "batch": 256, "fin": 9216, "mid": 4096, "fout": 4096},
        # a ResNet-18 stage: a large image, few channels, result bound by memory
        {"name": "conv_stage", "op": "conv", "n": 16, "c": 64, "h": 56, "w": 56, "o": 64, "k": 3, "stride": 1, "pad": 1,
         "out": "f32"},
        # a deep stage: small image, many channels
        {"name": "conv_deep", "op": "conv", "n": 64, "c": 256, "h": 14, "w": 14, "o": 256, "k": 3, "stride": 1, "pad": 1,
         "out": "f32"},
        # odd sizes all round: channels past a word, an uneven image, a stride that leaves a rest
        {"name": "conv_ragged", "op": "conv", "n": 7, "c": 130, "h": 29, "w": 27, "o": 70, "k": 3, "stride": 2, "pad": 1,
         "out": "i32"},
        # blocks of a binary network in a row without fp32 maps between them
        {"name": "conv_chain", "op": "conv_bits", "n": 16, "c": 64, "h": 56, "w": 56, "o": 64, "k": 3},
        # DoReFa: 2-bit activations, 1-bit weights
        {"name": "quant_2x1", "op": "quant", "m": 1024, "n": 1024, "k": 4096, "bits_a": 2, "bits_w": 1},
        # more bits on both sides, an uneven shape
        {"name": "quant_4x4", "op": "quant", "m": 500, "n": 1000, "k": 2304, "bits_a": 4, "bits_w": 4},
        # a product that fills the chip
        {"name": "gemm_large", "op": "gemm", "m": 8192, "n": 8192, "k": 8192, "word": 64, "count": False},
        # a classifier's weights on their way into a model file
        {"name": "convert_fc", "op": "convert", "kind": "fc", "o": 4096, "i": 9216},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, its logarithm spread evenly."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _size(rng, lo, hi):
    """A size of a layer: every other one a multiple of 64 as networks have them, the others as they come."""
    v = _log(rng, lo, hi)
    return v if rng.random() < 0.5 else max(64, v // 64 * 64)


def draw(rng):
    op = rng.choice(["fc", "fc_pair", "fc_bits", "conv", "conv_bits", "quant", "gemm", "convert"])
    if op == "fc":
        return {"op": op, "batch": _log(rng, 1, 1024), "fin": _size(rng, 64, 9216), "fout": _size(rng, 10, 4096),
                "out": rng.choice(["f32", "i32"])}
    if op in ("fc_pair", "fc_bits"):
        return {"op": op, "batch": _log(rng, 1, 1024), "fin": _size(rng, 256, 9216), "mid": _size(rng, 256, 4096),
                "fout": _size(rng, 10, 4096)}
    if op in ("conv", "conv_bits"):
        while True:
            k = rng.choice([1, 3, 3, 3, 5, 7]) if op == "conv" else rng.choice([3, 3, 3, 5])
            c = {"op": op, "n": _log(rng, 1, 200), "c": _size(rng, 16, 512), "h": _log(rng, 7, 56)}
            c.update(w=max(7, c["h"] + rng.choice([0, 0, -1, 2])), o=_size(rng, 16, 512), k=k)
            if op == "conv":
                c.update(stride=rng.choice([1, 1, 2]), pad=rng.choice([k // 2, k // 2, 0]), out=rng.choice(["f32", "f32", "i32"]))
            px = c["n"] * c["h"] * c["w"]
            if px * c["c"] <= 1 << 25 and px * c["o"] <= 1 << 24 and px * c["o"] * c["c"] * k * k <= 1 << 36:
                return c
    if op == "quant":
        while True:
            c = {"op": op, "m": _log(rng, 16, 2048), "n": _size(rng, 16, 2048), "k": _size(rng, 64, 8192),
                 "bits_a": rng.choice([1, 2, 2, 3, 4, 8]), "bits_w": rng.choice([1, 1, 2, 4, 8])}
            if c["m"] * c["n"] * c["k"] * c["bits_a"] * c["bits_w"] <= 1 << 35:
                return c
    if op == "gemm":
        return {"op": op, "m": _size(rng, 64, 8192), "n": _size(rng, 64, 8192), "k": _size(rng, 64, 8192),
                "word": rng.choice([64, 64, 32]), "count": rng.random() < 0.3}
    if rng.random() < 0.5:
        return {"op": op, "kind": rng.choice(["fc", "fc_in_out"]), "o": _size(rng, 64, 4096), "i": _size(rng, 64, 9216)}
    return {"op": op, "kind": "conv", "o": _size(rng, 16, 512), "c": _size(rng, 3, 512), "k": rng.choice([1, 3, 3, 5, 7])}


def _weights(g, *shape):
    return torch.empty(shape, device="cuda").uniform_(-1.0, 1.0, generator=g)


def _fc_layer(g, fin, fout):
    w = _weights(g, fout, fin)
    return B.binarize_pack(w, 1), B.alpha_mean_abs(w)


def _conv_layer(g, o, c, k):
    w = torch.randn((o, c, k, k), device="cuda", generator=g)
    return B.pack_conv_weights(w), B.alpha_mean_abs(w)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    op = case["op"]
    s = dict(case)
    if op == "fc":
        s["x"] = torch.randn((case["batch"], case["fin"]), device="cuda", generator=g)
        s["w"], s["alpha"] = _fc_layer(g, case["fin"], case["fout"])
    elif op in ("fc_pair", "fc_bits"):
        b, fin, mid, fout = case["batch"], case["fin"], case["mid"], case["fout"]
        s["x"] = torch.randn((b, fin), device="cuda", generator=g)
        s["w1"], s["alpha1"] = _fc_layer(g, fin, mid)
        s["w2"], s["alpha2"] = _fc_layer(g, mid, fout)
        if op == "fc_pair":  # a loop that keeps its buffers
            s["mid_out"] = torch.empty((b, mid), device="cuda")
            s["last"] = torch.empty((b, fout), device="cuda")
            need = max(B.workspace_bytes(B.OP_BINARY_FC, d) for d in ((b, fin, mid), (b, mid, fout)))
            s["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        else:
            s["thr"] = torch.randn(mid, device="cuda", generator=g) * (0.25 * math.sqrt(fin))
    elif op in ("conv", "conv_bits"):
        n, c, h, w, o, k = (case[v] for v in ("n", "c", "h", "w", "o", "k"))
        # what a ReLU and a shift leave: more than half of the signs positive
        s["x"] = torch.randn((n, c, h, w), device="cuda", generator=g).abs_().sub_(0.5)
        if op == "conv":
            s["w"], s["alpha"] = _conv_layer(g, o, c, k)
        else:
            s["layers"] = [_conv_layer(g, o, ci, k) for ci in (c, o, o)]
            s["thr"] = [torch.randn(o, device="cuda", generator=g) * (0.25 * k * math.sqrt(o)) for _ in range(2)]
    elif op == "quant":
        s["a"] = torch.rand((case["m"], case["k"]), device="cuda", generator=g)
        w = torch.randn((case["n"], case["k"]), device="cuda", generator=g)
        s["w"] = w if case["bits_w"] == 1 else torch.tanh(w)
    elif op == "gemm":
        wide = -(-case["k"] // case["word"])
        rest = case["k"] - (wide - 1) * case["word"]
        for name, rows in (("A", case["m"]), ("B", case["n"])):
            t = torch.randint(-2**31, 2**31, (rows, wide * case["word"] // 32), device="cuda", generator=g,
                              dtype=torch.int64).to(torch.int32)
            t = t.view(torch.int64) if case["word"] == 64 else t
            if rest < case["word"]:
                t[:, -1] &= (1 << rest) - 1
            s[name] = t
    else:
        shape = {"fc": ("o", "i"), "fc_in_out": ("i", "o"), "conv": ("o", "c", "k", "k")}[case["kind"]]
        s["w"] = _weights(g, *(case[v] for v in shape))
    return s


def run(s):
    op = s["op"]
    if op == "fc":
        if s["out"] == "i32":
            return B.binary_fc(s["x"], s["w"], integer_out=True)
        return B.binary_fc(s["x"], s["w"], alpha=s["alpha"])
    if op == "fc_pair":
        B.binary_fc(s["x"], s["w1"], alpha=s["alpha1"], out=s["mid_out"], workspace=s["workspace"])
        B.binary_fc(s["mid_out"], s["w2"], alpha=s["alpha2"], out=s["last"], workspace=s["workspace"])
        return [s["mid_out"], s["last"]]
    if op == "fc_bits":
        xp = B.binarize_pack(s["x"])
        mid = B.binary_fc_packed(xp, s["fin"], s["w1"], alpha=s["alpha1"], mode="bits", thr=s["thr"])
        return [mid, B.binary_fc_packed(mid, s["mid"], s["w2"], alpha=s["alpha2"])]
    if op == "conv":
        if s["out"] == "i32":
            return B.binary_conv2d(s["x"], s["w"], s["o"], s["k"], s["k"], s["stride"], s["pad"], integer_out=True)
        return B.binary_conv2d(s["x"], s["w"], s["o"], s["k"], s["k"], s["stride"], s["pad"], alpha=s["alpha"])
    if op == "conv_bits":
        k, o, pad = s["k"], s["o"], s["k"] // 2
        (w1, a1), (w2, a2), (w3, a3) = s["layers"]
        x0 = B.pack_nchw(s["x"], pad)
        x1 = B.binary_conv2d_bits(x0, s["c"], w1, o, k, k, 1, pad, alpha=a1, thr=s["thr"][0], out_pad=pad)
        x2 = B.binary_conv2d_bits(x1, o, w2, o, k, k, 1, pad, alpha=a2, thr=s["thr"][1], out_pad=pad)
        return [x1, x2, B.binary_conv2d_packed(x2, o, w3, o, k, k, 1, pad, alpha=a3)]
    if op == "quant":
        return B.quant_gemm(s["a"], s["w"], s["bits_a"], s["bits_w"], want_int=False)[1]
    if op == "gemm":
        if s["word"] == 32:
            return B.xnor_gemm_w32(s["A"], s["B"], s["k"])
        return B.xnor_gemm(s["A"], s["B"], s["k"], count=s["count"])
    if s["kind"] == "conv":
        return [B.pack_conv_weights(s["w"]), B.alpha_mean_abs(s["w"])]
    if s["kind"] == "fc_in_out":
        return B.binarize_pack(s["w"], 0)
    return [B.binarize_pack(s["w"], 1), B.alpha_mean_abs(s["w"])]


def work(case):
    """Bytes: fp32 and packed operands read once, results written once.  Flops: a multiply and an
    add for every (row, column, k), times the pairs of bit planes of a k-bit product."""
    op = case["op"]
    words = lambda k: 8 * (-(-k // 64))  # noqa: E731  bytes of a packed row
    if op == "fc":
        b, i, o = case["batch"], case["fin"], case["fout"]
        return {"bytes": 4 * b * i + o * words(i) + 4 * b * o, "flops": 2 * b * i * o}
    if op in ("fc_pair", "fc_bits"):
        b, i, m, o = case["batch"], case["fin"], case["mid"], case["fout"]
        return {"bytes": 4 * b * i + m * words(i) + o * words(m) + 4 * b * o + b * (4 * m if op == "fc_pair" else words(m)),
                "flops": 2 * b * (i * m + m * o)}
    if op in ("conv", "conv_bits"):
        n, c, h, w, o, k = (case[v] for v in ("n", "c", "h", "w", "o", "k"))
        if op == "conv":
            ho, wo = B.conv_out_hw(h, w, k, k, case["stride"], case["pad"])
            return {"bytes": 4 * n * c * h * w + o * k * k * words(c) + 4 * n * o * ho * wo, "flops": 2 * n * o * ho * wo * c * k * k}
        q = (h + 2 * (k // 2)) * (w + 2 * (k // 2))
        return {"bytes": 4 * n * c * h * w + o * k * k * (words(c) + 2 * words(o)) + 2 * n * q * words(o) + 4 * n * o * h * w,
                "flops": 2 * n * o * h * w * k * k * (c + 2 * o)}
    if op == "quant":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 4 * (m * k + n * k + m * n), "flops": 2 * m * n * k * case["bits_a"] * case["bits_w"]}
    if op == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": (m + n) * (-(-k // case["word"])) * case["word"] // 8 + 4 * m * n, "flops": 2 * m * n * k}
    o, i = case["o"], case["i"] if case["kind"] != "conv" else case["c"] * case["k"] ** 2
    return {"bytes": 4 * o * i + o * words(i) + (4 * o if case["kind"] != "fc_in_out" else 0), "flops": o * i}


def tolerance(case):
    """Bits and whole numbers are exact.  An fp32 result is a whole number scaled once, or a mean
    summed in 64 bits: the last bit of 24 at most."""
    op = case["op"]
    if op == "gemm" or case.get("out") == "i32" or case.get("kind") == "fc_in_out":
        return "exact"
    return {"rel": 1e-6}
