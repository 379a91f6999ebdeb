"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a plain dict.  `prepare` makes what a program holds before the call (inputs, weights, output buffers and the
tuned configurations, all on the GPU), `run` makes one pass through the public entry points, `work` and `tolerance` say
what a pass cannot do without and how far another correct implementation may be off, `exact` gives a pass's results in 64 bits.

Kinds of cases and what they stand for:
  gemm        one GEMM with its fused epilogue (optionally with a residual matrix), tuned or left to the built-in rule
  gemm_pair   two GEMMs fused back to back: the recommendation-model pairs of the paper's Table 1
  gemm_chain  three GEMMs fused back to back
  conv_pair   a convolution and the 1x1 behind it, fused: the pairs of Table 2 and the fused tail of a bottleneck
  unpadded    a convolution whose channel count is even but no multiple of 8 (Table 3), called without padding it
  block       one residual bottleneck block in two launches: 1x1, then 3x3 -> 1x1 + skip connection + ReLU
  resnet      the convolutions of a ResNet-50 behind its stem, in order, each layer reading what the last one wrote
  image       the edges of a network: the image (NCHW, 3 channels) into the first layer, a feature map back to NCHW
"""
import math

import torch

import paper_2110_15238_amd as bolt

ACTS = ("none", "relu", "gelu", "hardswish", "softplus")


def listed():
    return [
        # The smallest call: one 256^3 GEMM + bias + ReLU as it is made without tuning first; launch and call bound.
        dict(name="gemm_small", kind="gemm", M=256, N=256, K=256, layout="kn", act="relu", residual=False, tuned=False),
        # The classifier behind a ResNet-50 at batch 32: few rows, a deep reduction, an odd width; no activation.
        dict(name="gemm_head", kind="gemm", M=32, N=1000, K=2048, layout="kn", act="none", residual=False, tuned=True),
        # The paper's epilogue-fusion GEMM (Section 4.1.1, a transformer MLP's first half) with GELU.
        dict(name="gemm_mlp", kind="gemm", M=1280, N=3072, K=768, layout="kn", act="gelu", residual=False, tuned=True),
        # The largest: a GEMM that fills the chip for many tiles per compute unit, weights as [N][K].
        dict(name="gemm_large", kind="gemm", M=8192, N=8192, K=8192, layout="nk", act="relu", residual=False, tuned=True),
        # Table 1, row 3: 32768 rows, 576 -> 128 -> 64, row-major weights.
        dict(name="gemm_pair", kind="gemm_pair", M=32768, K0=576, N0=128, N1=64, layout="kn", act="relu"),
        # A chain of three thin GEMMs over many rows (the widths of Table 1, row 4, with its first op repeated).
        dict(name="gemm_chain", kind="gemm_chain", M=128320, K0=96, N0=32, N1=96, N2=32, layout="kn", act="relu"),
        # 3x3 64 -> 64, then 1x1 64 -> 256, at batch 32: the tail of a first-stage bottleneck without its skip.
        dict(name="conv_pair", kind="conv_pair", batch=32, H=56, W=56, C=64, K0=64, R=3, stride=1, K1=256),
        # Table 3, row 3: 46 input channels, a 5x7 filter, no padding of the image or of the channels.
        dict(name="conv_unpadded", kind="unpadded", batch=128, H=14, W=19, C=46, K=32, R=5, S=7, pad_h=0, pad_w=0),
        # A residual bottleneck block of the first stage at batch 32.
        dict(name="block", kind="block", batch=32, H=56, W=56, mid=64, out=256),
        # The network's body for one image (latency: many small launches) and for a batch of 32 (throughput).
        dict(name="resnet_b1", kind="resnet", batch=1, hw=56),
        dict(name="resnet_b32", kind="resnet", batch=32, hw=56),
        # 32 images of 224 x 224 into the 7x7/2 first layer as they come (NCHW), and the first stage's output handed
        # back to an NCHW consumer.
        dict(name="image_edges", kind="image", batch=32, H=224, W=224, K=64, R=7, out_hw=56, out_c=256),
    ]


# ----------------------------------------------------------------------------------------------------------------
# draws from the same ranges
# ----------------------------------------------------------------------------------------------------------------
def _log(rng, lo, hi, step=1):
    """An integer in [lo, hi], its logarithm uniform, rounded to a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def _draw_gemm(rng):
    while True:
        c = dict(kind="gemm", M=_log(rng, 1, 8192), N=_log(rng, 16, 8192, 8), K=_log(rng, 64, 8192, 8),
                 layout=rng.choice(("kn", "nk")), act=rng.choice(ACTS), residual=rng.random() < 0.25,
                 tuned=rng.random() < 0.7)
        if 2 * c["M"] * c["N"] * c["K"] <= 2 * 8192 ** 3:
            return c


def _draw_gemm_pair(rng):
    n0, n1 = rng.choice(((64, 256), (128, 128)))
    return dict(kind="gemm_pair", M=_log(rng, 1000, 131072), K0=_log(rng, 8, 576, 8), N0=_log(rng, 8, n0, 8),
                N1=_log(rng, 8, n1, 8), layout=rng.choice(("kn", "nk")), act=rng.choice(("relu", "relu", "gelu", "hardswish")))


def _draw_gemm_chain(rng):
    while True:
        c = dict(kind="gemm_chain", M=_log(rng, 1000, 131072), K0=_log(rng, 32, 576, 8), N0=_log(rng, 16, 128, 8),
                 N1=_log(rng, 16, 128, 8), N2=_log(rng, 16, 128, 8), layout=rng.choice(("kn", "nk")),
                 act=rng.choice(("relu", "relu", "gelu", "hardswish")))
        op = bolt.OP_GEMM_CHAIN3
        if bolt.bolt_check_chain(op, _chain_descs(c)) == 0:  # the widths fit a compiled chain
            return c


def _draw_conv_pair(rng):
    r = rng.choice((1, 3, 3))
    stride = rng.choice((1, 1, 2))
    hw = rng.randint(14, 112)
    most = max(1, min(64, int(32 * 112 * 112 / (hw * hw))))
    return dict(kind="conv_pair", batch=_log(rng, 1, most), H=hw, W=hw, C=_log(rng, 16, 128, 8), K0=_log(rng, 24, 64, 8),
                R=r, stride=stride, K1=_log(rng, 32, 256, 8))


def _draw_unpadded(rng):
    r, s = rng.choice(((3, 3), (5, 5), (5, 7)))
    pad = rng.random() < 0.6
    c = _log(rng, 10, 174, 2)
    return dict(kind="unpadded", batch=_log(rng, 8, 288), H=rng.randint(11, 20), W=rng.randint(14, 26),
                C=c if c % 8 else c + 2, K=_log(rng, 16, 64, 8), R=r, S=s, pad_h=r // 2 if pad else 0, pad_w=s // 2 if pad else 0)


def _draw_block(rng):
    mid = rng.choice((32, 40, 48, 56, 64))
    return dict(kind="block", batch=_log(rng, 1, 32), H=rng.randint(20, 56), W=rng.randint(20, 56), mid=mid, out=4 * mid)


def _draw_resnet(rng):
    return dict(kind="resnet", batch=_log(rng, 1, 32), hw=rng.randint(32, 56))


def _draw_image(rng):
    hw = rng.randint(96, 224)
    return dict(kind="image", batch=_log(rng, 1, 32), H=hw, W=hw, K=rng.choice((32, 48, 64)), R=rng.choice((3, 7)),
                out_hw=rng.choice((7, 14, 28, 56)), out_c=rng.choice((64, 256, 512, 1000)))


def draw(rng):
    kinds = (_draw_gemm, _draw_gemm, _draw_gemm, _draw_gemm_pair, _draw_gemm_chain, _draw_conv_pair, _draw_unpadded,
             _draw_block, _draw_resnet, _draw_resnet, _draw_image)
    return rng.choice(kinds)(rng)


# ----------------------------------------------------------------------------------------------------------------
# what a program holds before the call
# ----------------------------------------------------------------------------------------------------------------
_untuned = False  # set while exact() makes the inputs: it has no use for a configuration


class _Make:
    """Seeded tensors.  Activations are U[-1, 1] (behind a ReLU where `relu`), weights N(0, 2 / fan_in), biases small."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(int(seed) * 7919 + 17)

    def x(self, *shape, relu=False):
        t = torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-1, 1, generator=self.gen)
        return (t.clamp_(min=0) if relu else t).half()

    def w(self, *shape, fan_in, scale=1.0):
        t = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0, scale * math.sqrt(2 / fan_in), generator=self.gen)
        return t.half()

    def b(self, n):
        return torch.empty(n, dtype=torch.float32, device="cuda").uniform_(-0.5, 0.5, generator=self.gen).half()

    @staticmethod
    def out(*shape):
        return torch.empty(shape, dtype=torch.float16, device="cuda")


def _tuned(op, d0, d1, tensors):
    """The configuration a program keeps for a problem, and the workspace it needs (None if it needs none)."""
    if _untuned:
        return None, None
    most = bolt.bolt_workspace_bytes(op, d0, d1)
    scratch = torch.empty(most, dtype=torch.uint8, device="cuda") if most else None
    config = bolt.bolt_tune(op, d0, d1, tensors, scratch).config
    need = bolt.bolt_workspace_bytes(op, d0, d1, config)
    return config, torch.empty(need, dtype=torch.uint8, device="cuda") if need else None


def _layout(c):
    return bolt.LAYOUT_KN if c["layout"] == "kn" else bolt.LAYOUT_NK


def _weight(make, c, k, n, scale=1.0):
    return make.w(*((k, n) if c["layout"] == "kn" else (n, k)), fan_in=k, scale=scale)


def _chain_descs(c):
    m, lay = c["M"], _layout(c)
    widths = [c["K0"], c["N0"], c["N1"], c["N2"]]
    return [bolt.gemm_desc(m, n, k, act=c["act"], b_layout=lay) for k, n in zip(widths, widths[1:])]


def _prepare_gemm(c, make):
    d = bolt.gemm_desc(c["M"], c["N"], c["K"], act=c["act"], b_layout=_layout(c))
    a, w, b, y = make.x(c["M"], c["K"]), _weight(make, c, c["K"], c["N"]), make.b(c["N"]), make.out(c["M"], c["N"])
    kw = {}
    if c["tuned"]:
        kw["config"], kw["workspace"] = _tuned(bolt.OP_GEMM, d, None, [a, w, b, y])
    if c["residual"]:
        skip = make.x(c["M"], c["N"])
        return [(bolt.bolt_gemm_epilogue_residual, (d, a, w, b, skip, y), kw)], [y]
    return [(bolt.bolt_gemm_epilogue, (d, a, w, b, y), kw)], [y]


def _prepare_gemm_pair(c, make):
    m, lay = c["M"], _layout(c)
    g0 = bolt.gemm_desc(m, c["N0"], c["K0"], act=c["act"], b_layout=lay)
    g1 = bolt.gemm_desc(m, c["N1"], c["N0"], act=c["act"], b_layout=lay)
    args = [make.x(m, c["K0"]), _weight(make, c, c["K0"], c["N0"]), make.b(c["N0"]), _weight(make, c, c["N0"], c["N1"]),
            make.b(c["N1"]), make.out(m, c["N1"])]
    config, _ = _tuned(bolt.OP_B2B_GEMM, g0, g1, args)
    return [(bolt.bolt_b2b_gemm, (g0, g1, *args), dict(config=config))], [args[-1]]


def _prepare_gemm_chain(c, make):
    descs = _chain_descs(c)
    widths = [c["K0"], c["N0"], c["N1"], c["N2"]]
    a = make.x(c["M"], c["K0"])
    ws = [_weight(make, c, k, n) for k, n in zip(widths, widths[1:])]
    bs = [make.b(n) for n in widths[1:]]
    y = make.out(c["M"], c["N2"])
    config = bolt.bolt_tune_chain(bolt.OP_GEMM_CHAIN3, descs, [a, ws[0], bs[0], ws[1], bs[1], ws[2], bs[2], y]).config
    return [(bolt.bolt_b2b_gemm_chain, (descs, a, ws, bs, y), dict(config=config))], [y]


def _prepare_conv_pair(c, make):
    n, h, w_, r = c["batch"], c["H"], c["W"], c["R"]
    c0 = bolt.conv_desc(n, h, w_, c["C"], c["K0"], r, r, c["stride"], r // 2)
    p, q = bolt.conv_out_hw(c0)
    c1 = bolt.conv_desc(n, p, q, c["K0"], c["K1"], 1, 1)
    args = [make.x(n, h, w_, c["C"], relu=True), make.w(c["K0"], r, r, c["C"], fan_in=r * r * c["C"]), make.b(c["K0"]),
            make.w(c["K1"], 1, 1, c["K0"], fan_in=c["K0"]), make.b(c["K1"]), make.out(n, p, q, c["K1"])]
    config, _ = _tuned(bolt.OP_B2B_CONV, c0, c1, args)
    return [(bolt.bolt_b2b_conv, (c0, c1, *args), dict(config=config))], [args[-1]]


def _prepare_unpadded(c, make):
    d = bolt.conv_desc(c["batch"], c["H"], c["W"], c["C"], c["K"], c["R"], c["S"], 1, (c["pad_h"], c["pad_w"]))
    p, q = bolt.conv_out_hw(d)
    x, b = make.x(c["batch"], c["H"], c["W"], c["C"], relu=True), make.b(c["K"])
    w = make.w(c["K"], c["R"], c["S"], c["C"], fan_in=c["R"] * c["S"] * c["C"])
    y = make.out(c["batch"], p, q, c["K"])
    config, ws = _tuned(bolt.OP_CONV2D, d, None, [x, w, b, y])
    return [(bolt.bolt_conv2d_fprop_nhwc, (d, x, w, b, y), dict(config=config, workspace=ws))], [y]


def _conv(make, x, k, r, stride, act="relu", y=None, skip=None, scale=1.0):
    """One tuned convolution (pad r // 2) on tensor x: its call and its output."""
    n, h, w_, ch = x.shape
    d = bolt.conv_desc(n, h, w_, ch, k, r, r, stride, r // 2, act=act)
    w, b = make.w(k, r, r, ch, fan_in=r * r * ch, scale=scale), make.b(k)
    y = make.out(n, *bolt.conv_out_hw(d), k) if y is None else y
    config, ws = _tuned(bolt.OP_CONV2D, d, None, [x, w, b, y])
    kw = dict(config=config, workspace=ws)
    if skip is None:
        return (bolt.bolt_conv2d_fprop_nhwc, (d, x, w, b, y), kw), y
    return (bolt.bolt_conv2d_fprop_nhwc_residual, (d, x, w, b, skip, y), kw), y


def _prepare_block(c, make):
    n, h, w_, mid, out = c["batch"], c["H"], c["W"], c["mid"], c["out"]
    x = make.x(n, h, w_, out, relu=True)
    first, t = _conv(make, x, mid, 1, 1)
    c0 = bolt.conv_desc(n, h, w_, mid, mid, 3, 3, 1, 1)
    c1 = bolt.conv_desc(n, h, w_, mid, out, 1, 1)
    w0, b0 = make.w(mid, 3, 3, mid, fan_in=9 * mid), make.b(mid)
    w1, b1 = make.w(out, 1, 1, mid, fan_in=mid, scale=0.5), make.b(out)
    y = make.out(n, h, w_, out)
    config, _ = _tuned(bolt.OP_B2B_CONV_RES, c0, c1, [t, w0, b0, w1, b1, y, x])
    return [first, (bolt.bolt_b2b_conv_residual, (c0, c1, t, w0, b0, w1, b1, x, y), dict(config=config))], [y]


# blocks, bottleneck width, output width and stride of the four stages of a ResNet-50 (the stride is on the 3x3)
_STAGES = ((3, 64, 256, 1), (4, 128, 512, 2), (6, 256, 1024, 2), (3, 512, 2048, 2))


def _prepare_resnet(c, make):
    x = make.x(c["batch"], c["hw"], c["hw"], 64, relu=True)  # what the stem and its pooling hand over
    calls, outputs = [], []
    for blocks, mid, out, stride in _STAGES:
        for i in range(blocks):
            s = stride if i == 0 else 1
            skip = x
            if i == 0:
                call, skip = _conv(make, x, out, 1, s, act="none")
                calls.append(call)
            call, t = _conv(make, x, mid, 1, 1)
            calls.append(call)
            call, t = _conv(make, t, mid, 3, s)
            calls.append(call)
            call, x = _conv(make, t, out, 1, 1, skip=skip, scale=0.25)
            calls.append(call)
        outputs.append(x)  # the feature maps of the four stages
    return calls, outputs


def _prepare_image(c, make):
    n, h, w_, k, r = c["batch"], c["H"], c["W"], c["K"], c["R"]
    d = bolt.conv_desc(n, h, w_, 3, k, r, r, 2, r // 2, x_layout="nchw")
    x, w, b = make.x(n, 3, h, w_), make.w(k, r, r, 3, fan_in=r * r * 3), make.b(k)
    y = make.out(n, *bolt.conv_out_hw(d), k)
    config, ws = _tuned(bolt.OP_CONV2D, d, None, [x, w, b, y])
    f = make.x(n, c["out_hw"], c["out_hw"], c["out_c"], relu=True)
    g = make.out(n, c["out_c"], c["out_hw"], c["out_hw"])
    return [(bolt.bolt_conv2d_fprop_nhwc, (d, x, w, b, y), dict(config=config, workspace=ws)),
            (bolt.bolt_nhwc_to_nchw, (f, g), {})], [y, g]


_PREPARE = dict(gemm=_prepare_gemm, gemm_pair=_prepare_gemm_pair, gemm_chain=_prepare_gemm_chain, conv_pair=_prepare_conv_pair,
                unpadded=_prepare_unpadded, block=_prepare_block, resnet=_prepare_resnet, image=_prepare_image)


def prepare(case, seed):
    calls, outputs = _PREPARE[case["kind"]](case, _Make(seed))
    return dict(calls=calls, outputs=outputs)


def run(state):
    for call, args, kwargs in state["calls"]:
        call(*args, **kwargs)
    return state["outputs"]


# ----------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ----------------------------------------------------------------------------------------------------------------
def _conv_work(n, h, w, c, k, r, s, stride, ph, pw, skip=False):
    """(bytes, flops, P, Q) of one convolution: each tensor once; a strided 1x1 only the pixels it samples."""
    p, q = (h + 2 * ph - r) // stride + 1, (w + 2 * pw - s) // stride + 1
    pixels = n * p * q if r == 1 and s == 1 else n * h * w
    halves = pixels * c + k * r * s * c + k + n * p * q * k * (2 if skip else 1)
    return 2 * halves, 2 * n * p * q * k * r * s * c, p, q


def work(case):
    c, kind = case, case["kind"]
    if kind == "gemm":
        m, n, k = c["M"], c["N"], c["K"]
        return dict(bytes=2 * (m * k + k * n + n + m * n * (2 if c["residual"] else 1)), flops=2 * m * n * k)
    if kind in ("gemm_pair", "gemm_chain"):
        w = [c["K0"], c["N0"], c["N1"]] + ([c["N2"]] if kind == "gemm_chain" else [])
        macs = sum(a * b for a, b in zip(w, w[1:]))
        return dict(bytes=2 * (c["M"] * (w[0] + w[-1]) + macs + sum(w[1:])), flops=2 * c["M"] * macs)
    if kind == "unpadded":
        b, f, _, _ = _conv_work(c["batch"], c["H"], c["W"], c["C"], c["K"], c["R"], c["S"], 1, c["pad_h"], c["pad_w"])
        return dict(bytes=b, flops=f)
    if kind == "conv_pair":
        b, f, p, q = _conv_work(c["batch"], c["H"], c["W"], c["C"], c["K0"], c["R"], c["R"], c["stride"], c["R"] // 2, c["R"] // 2)
        m = c["batch"] * p * q
        return dict(bytes=b + 2 * (m * (c["K1"] - c["K0"]) + c["K0"] * c["K1"] + c["K1"]), flops=f + 2 * m * c["K0"] * c["K1"])
    if kind == "block":
        n, h, w, mid, out = c["batch"], c["H"], c["W"], c["mid"], c["out"]
        m = n * h * w
        b0, f0, _, _ = _conv_work(n, h, w, out, mid, 1, 1, 1, 0, 0)
        halves = m * mid + 9 * mid * mid + mid + mid * out + out + 2 * m * out
        return dict(bytes=b0 + 2 * halves, flops=f0 + 2 * m * (9 * mid * mid + mid * out))
    if kind == "resnet":
        n, h, ch, total_b, total_f = c["batch"], c["hw"], 64, 0, 0
        for blocks, mid, out, stride in _STAGES:
            for i in range(blocks):
                s = stride if i == 0 else 1
                parts = [_conv_work(n, h, h, ch, out, 1, 1, s, 0, 0)] if i == 0 else []
                parts += [_conv_work(n, h, h, ch, mid, 1, 1, 1, 0, 0), _conv_work(n, h, h, mid, mid, 3, 3, s, 1, 1)]
                h, ch = parts[-1][2], out
                parts.append(_conv_work(n, h, h, mid, out, 1, 1, 1, 0, 0, skip=True))
                total_b += sum(x[0] for x in parts)
                total_f += sum(x[1] for x in parts)
        return dict(bytes=total_b, flops=total_f)
    b, f, _, _ = _conv_work(c["batch"], c["H"], c["W"], 3, c["K"], c["R"], c["R"], 2, c["R"] // 2, c["R"] // 2)
    return dict(bytes=b + 4 * c["batch"] * c["out_hw"] ** 2 * c["out_c"], flops=f)


# ----------------------------------------------------------------------------------------------------------------
# the same pass in 64 bits
# ----------------------------------------------------------------------------------------------------------------
def _act64(v, act):
    name = {number: text for text, number in bolt.ACT.items()}[act]
    if name == "relu":
        return v.clamp_(min=0)
    if name == "gelu":
        return 0.5 * v * torch.erfc(v * -math.sqrt(0.5))
    if name == "hardswish":
        return v * (v + 3).clamp_(0, 6) / 6
    return torch.logaddexp(v, torch.zeros((), dtype=v.dtype, device=v.device)) if name == "softplus" else v


def _gemm64(d, a, w, b, skip=None):
    v = a @ (w.double() if d.b_layout == bolt.LAYOUT_KN else w.double().t()) + b.double()
    return _act64(v if skip is None else v + skip.double(), d.act)


def _conv64(d, x, w, b, skip=None):
    """x: NHWC, 64 bits.  Each filter tap is a matrix product over the pixels that it meets."""
    p, q = (d.H + 2 * d.pad_h - d.R) // d.stride_h + 1, (d.W + 2 * d.pad_w - d.S) // d.stride_w + 1
    x = torch.nn.functional.pad(x, (0, 0, d.pad_w, d.pad_w, d.pad_h, d.pad_h))
    v = b.double().expand(d.N * p * q, d.K).clone()
    for r in range(d.R):
        for s in range(d.S):
            tap = x[:, r:r + (p - 1) * d.stride_h + 1:d.stride_h, s:s + (q - 1) * d.stride_w + 1:d.stride_w]
            v.addmm_(tap.reshape(-1, d.C), w[:, r, s].double().t())
    v = v.view(d.N, p, q, d.K)
    return _act64(v if skip is None else v + skip, d.act)


def exact(case, seed):
    """What `run` returns, in 64 bits from the same half inputs; nothing is rounded between two ops."""
    global _untuned
    _untuned = True
    try:
        calls, outputs = _PREPARE[case["kind"]](case, _Make(seed))
    finally:
        _untuned = False
    have = {}  # results so far, by the address of the buffer that the pass writes them to

    def get(t):
        return have.get(t.data_ptr(), t)

    for call, a, _ in calls:
        if call is bolt.bolt_gemm_epilogue:
            out, v = a[4], _gemm64(a[0], a[1].double(), a[2], a[3])
        elif call is bolt.bolt_gemm_epilogue_residual:
            out, v = a[5], _gemm64(a[0], a[1].double(), a[2], a[3], a[4])
        elif call is bolt.bolt_b2b_gemm:
            out, v = a[7], _gemm64(a[1], _gemm64(a[0], a[2].double(), a[3], a[4]), a[5], a[6])
        elif call is bolt.bolt_b2b_gemm_chain:
            out, v = a[4], a[1].double()
            for d, w, b in zip(a[0], a[2], a[3]):
                v = _gemm64(d, v, w, b)
        elif call is bolt.bolt_conv2d_fprop_nhwc:
            x = get(a[1]).double()
            out, v = a[4], _conv64(a[0], x.permute(0, 2, 3, 1) if a[0].x_layout == bolt.TENSOR_NCHW else x, a[2], a[3])
        elif call is bolt.bolt_conv2d_fprop_nhwc_residual:
            out, v = a[5], _conv64(a[0], get(a[1]).double(), a[2], a[3], get(a[4]).double())
        elif call is bolt.bolt_b2b_conv:
            out, v = a[7], _conv64(a[1], _conv64(a[0], get(a[2]).double(), a[3], a[4]), a[5], a[6])
        elif call is bolt.bolt_b2b_conv_residual:
            out, v = a[8], _conv64(a[1], _conv64(a[0], get(a[2]).double(), a[3], a[4]), a[5], a[6], get(a[7]).double())
        else:
            out, v = a[1], get(a[0]).double().permute(0, 3, 1, 2).contiguous()
        have[out.data_ptr()] = v
    return [have[t.data_ptr()] for t in outputs]


def tolerance(case):
    # Outputs are halves, sums are 32 bits wide: one rounding of the result, and one of each tensor between two ops.
    # Against the same passes in 64 bits (operands and constants as halves in memory, nothing rounded in between) single
    # ops are off by 2.2e-4, pairs by 3.0e-4, chains of three by 4.0e-4, the block by 2.5e-4 and the last feature map of
    # the network by 7.0e-4; stated is about four times that.
    return {"rel": {"gemm": 9e-4, "gemm_pair": 1.2e-3, "gemm_chain": 1.6e-3, "conv_pair": 1.2e-3, "unpadded": 9e-4, "block": 1.0e-3,
                    "resnet": 2.8e-3, "image": 9e-4}[case["kind"]]}
