"""What users of this library have it do, as cases that can be timed and whose outputs can be compared.

A training program keeps, per layer, 8-bit codes with their quantizers, range states and statistics in
device memory and calls the entry points of ``paper_2105_04246_amd`` on them; ``run`` below is one such
pass.  Shapes are those of this repository's own networks and tests (ResNet-18-, VGG16- and
MobileNetV2-shaped layers, linear layers, element-wise tensors) or generic ones; values follow the
distributions the paper describes (post-ReLU activations, He-normal weights, Laplace gradients with
outliers) and are drawn on the GPU from the seed alone.

Kinds of case
  layer    forward, input gradient, weight gradient and both range updates of one layer
  network  the same over a stack of layers (``passes`` = "step"), or its forward pass and the range
           updates alone ("forward")
  tensor   quantization of an FP32 tensor that no GEMM of the library produced
  weights  quantization and re-laying of all weights of a network after an optimizer update
"""
import math
from collections import namedtuple

import torch

import paper_2105_04246_amd as hq

Layer = namedtuple("Layer", "kind B H W C R S stride pad Cout")
LINEAR, CONV, DEPTHWISE = hq.HQ_LINEAR, hq.HQ_CONV2D, hq.HQ_DEPTHWISE


# ---------------------------------------------------------------------------------------
# layer shapes
# ---------------------------------------------------------------------------------------

def _conv(B, H, W, C, k, stride, Cout):
    return Layer(CONV, B, H, W, C, k, k, stride, k // 2, Cout)


def _out_hw(L):
    return (L.H + 2 * L.pad - L.R) // L.stride + 1, (L.W + 2 * L.pad - L.S) // L.stride + 1


def _in_elems(L):
    return L.B * L.H * L.W * L.C


def _out_elems(L):
    oh, ow = _out_hw(L)
    return L.B * oh * ow * L.Cout


def _w_elems(L):
    return L.R * L.S * L.C * (1 if L.kind == DEPTHWISE else L.Cout)


def _macs(L):
    return _out_elems(L) * L.R * L.S * (1 if L.kind == DEPTHWISE else L.C)


def _resnet18(B, image):
    """3-channel 7x7/2 stem, four stages of 3x3 layers with 1x1 stride-2 shortcuts, 1000 classes."""
    layers = [_conv(B, image, image, 3, 7, 2, 64)]
    s = (_out_hw(layers[0])[0] + 1) // 2                       # 3x3 stride-2 pooling
    layers += [_conv(B, s, s, 64, 3, 1, 64) for _ in range(4)]
    cin = 64
    for cout in (128, 256, 512):
        layers += [_conv(B, s, s, cin, 3, 2, cout), _conv(B, s, s, cin, 1, 2, cout)]
        s = (s + 1) // 2
        layers += [_conv(B, s, s, cout, 3, 1, cout) for _ in range(3)]
        cin = cout
    return layers + [Layer(LINEAR, B, 1, 1, 512, 1, 1, 1, 0, 1000)]


def _vgg16(B, image):
    """13 3x3 layers in five blocks with 2x2 pooling between them, three linear layers, 200 classes."""
    layers, cin, s = [], 3, image
    for cout, n in ((64, 2), (128, 2), (256, 3), (512, 3), (512, 3)):
        for _ in range(n):
            layers.append(_conv(B, s, s, cin, 3, 1, cout))
            cin = cout
        s //= 2
    dims = (cin * s * s, 4096, 4096, 200)
    return layers + [Layer(LINEAR, B, 1, 1, k, 1, 1, 1, 0, n) for k, n in zip(dims, dims[1:])]


def _inverted_residual(B, hw, cin, cout, stride):
    """MobileNetV2 block: 1x1 expansion by 6, 3x3 depthwise, 1x1 projection."""
    mid = 6 * cin
    dw = Layer(DEPTHWISE, B, hw, hw, mid, 3, 3, stride, 1, mid)
    oh, ow = _out_hw(dw)
    return [_conv(B, hw, hw, cin, 1, 1, mid), dw, _conv(B, oh, ow, mid, 1, 1, cout)]


def _layers(case):
    if case["kind"] == "layer":
        return [Layer({"linear": LINEAR, "conv": CONV, "depthwise": DEPTHWISE}[case["op"]],
                      *(case[f] for f in Layer._fields[1:]))]
    if case["network"] == "resnet18":
        return _resnet18(case["B"], case["image"])
    if case["network"] == "vgg16":
        return _vgg16(case["B"], case["image"])
    return _inverted_residual(case["B"], case["image"], case["cin"], case["cout"], case["stride"])


def _layer_case(L, rounding, ranges, **more):
    return dict(more, kind="layer", op={LINEAR: "linear", CONV: "conv", DEPTHWISE: "depthwise"}[L.kind],
                rounding=rounding, ranges=ranges, **{f: getattr(L, f) for f in Layer._fields[1:]})


def listed():
    net = dict(kind="network", rounding="nearest", passes="step")
    return [
        # the smallest call: one linear layer of a small network, where launches and the host count
        _layer_case(Layer(LINEAR, 256, 1, 1, 512, 1, 1, 1, 0, 512), "nearest", "in-hindsight", name="linear_256x512x512"),
        # ranges calibrated on single images: a forward pass at batch 1, latency-bound
        dict(net, name="resnet18_forward_b1", network="resnet18", B=1, image=224, passes="forward"),
        # the ordinary large layer: ResNet stage 1 at batch 128
        _layer_case(_conv(128, 56, 56, 64, 3, 1, 64), "nearest", "in-hindsight", name="conv3x3_64_56_b128"),
        # ResNet stage 2 as the paper trains it, activation gradients rounded stochastically
        _layer_case(_conv(128, 28, 28, 128, 3, 1, 128), "stochastic", "in-hindsight", name="conv3x3_128_28_b128_sr"),
        # the same large layer under the dynamic two-pass estimator, for users who compare the two
        _layer_case(_conv(128, 56, 56, 64, 3, 1, 64), "nearest", "current", name="conv3x3_64_56_b128_dynamic"),
        # nothing aligned: odd image sides, channel counts that are multiples of 4 only, stride 2, odd batch
        _layer_case(Layer(CONV, 17, 29, 23, 36, 3, 3, 2, 1, 100), "nearest", "in-hindsight", name="conv3x3_ragged"),
        # point-wise and depthwise layers, bound by memory and by the epilogue
        dict(net, name="mobilenetv2_block_b128", network="inverted_residual", B=128, image=56, cin=32, cout=32, stride=1),
        # a whole step on small images at a small batch: many short launches
        dict(net, name="resnet18_64px_b32_sr", network="resnet18", B=32, image=64, rounding="stochastic"),
        # a whole step of the paper's Tiny ImageNet runs
        dict(net, name="vgg16_64px_b128_sr", network="vgg16", B=128, image=64, rounding="stochastic"),
        # the largest: a whole ImageNet-sized step at batch 256
        dict(net, name="resnet18_224px_b256", network="resnet18", B=256, image=224),
        # the output of a normalisation layer, quantized with the range of earlier iterations
        dict(name="tensor_activation_25m", kind="tensor", n=128 * 56 * 56 * 64, mode="in-hindsight", values="activation"),
        # all weights of a network after an optimizer update
        dict(name="weights_resnet18", kind="weights", network="resnet18", B=1, image=224),
    ]


# ---------------------------------------------------------------------------------------
# further cases of the same ranges
# ---------------------------------------------------------------------------------------

def _log_int(rng, lo, hi, multiple=1):
    """A multiple of `multiple` in lo..hi, uniform over the logarithm."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(-(-lo // multiple), min(hi // multiple, round(x / multiple))) * multiple


def _fit(L, most_macs=40e9, most_elems=200e6):
    """The layer with its batch reduced until one of its operations stays inside the limits."""
    per = max(_macs(L._replace(B=1)) / most_macs, max(_in_elems(L._replace(B=1)), _out_elems(L._replace(B=1))) / most_elems)
    return L._replace(B=max(1, min(L.B, int(1 / per))))


def _draw_layer(rng):
    family = rng.choice(("linear", "body", "body", "pointwise", "depthwise", "ragged", "first"))
    B, hw = _log_int(rng, 1, 256), _log_int(rng, 7, 112)
    if family == "linear":
        L = Layer(LINEAR, _log_int(rng, 1, 8192), 1, 1, _log_int(rng, 64, 4096, 4), 1, 1, 1, 0, _log_int(rng, 16, 4096, 4))
    elif family == "body":
        C = _log_int(rng, 64, 512, 64)
        L = _conv(B, hw, hw, C, 3, rng.choice((1, 1, 1, 2)), rng.choice((C, C, min(512, 2 * C))))
    elif family == "pointwise":
        L = _conv(B, hw, hw, _log_int(rng, 16, 960, 8), 1, rng.choice((1, 1, 2)), _log_int(rng, 16, 960, 8))
    elif family == "depthwise":
        C = _log_int(rng, 16, 960, 8)
        L = Layer(DEPTHWISE, B, hw, hw, C, 3, 3, rng.choice((1, 1, 2)), 1, C)
    elif family == "ragged":
        L = _conv(min(B, 64), hw, _log_int(rng, 7, 112), _log_int(rng, 4, 256, 4), rng.choice((1, 3, 3, 5)),
                  rng.choice((1, 2)), _log_int(rng, 4, 256, 4))
    else:
        k, stride = rng.choice(((7, 2), (3, 1), (3, 2)))
        side = _log_int(rng, 32, 224)
        L = _conv(B, side, side, 3, k, stride, 16 * rng.randint(1, 4))
    return _fit(L)


def draw(rng):
    what = rng.choice(("layer",) * 6 + ("dynamic", "network", "network", "tensor", "tensor", "weights"))
    rounding = rng.choice(("nearest", "stochastic"))
    if what == "layer":
        return _layer_case(_draw_layer(rng), rounding, "in-hindsight")
    if what == "dynamic":
        return _layer_case(_fit(_draw_layer(rng), most_elems=100e6), rounding, rng.choice(("current", "running")))
    if what == "network":
        network = rng.choice(("resnet18", "vgg16", "inverted_residual"))
        case = dict(kind="network", network=network, rounding=rounding, passes=rng.choice(("step", "step", "forward")))
        if network == "inverted_residual":
            cin = _log_int(rng, 16, 160, 8)
            case.update(image=_log_int(rng, 7, 112), cin=cin, cout=_log_int(rng, cin, 160, 8), stride=rng.choice((1, 1, 2)))
            at_one = sum(_in_elems(L) + _out_elems(L) for L in _layers(dict(case, B=1)))
            most = int(600e6 / at_one)
        else:
            case["image"] = 32 * rng.randint(1, 7)
            at_one = sum(_macs(L) for L in _layers(dict(case, B=1)))
            most = int(0.9 * sum(map(_macs, _resnet18(256, 224))) / at_one)
        case["B"] = _log_int(rng, 1, max(1, min(256, most)))
        return case
    if what == "tensor":
        return dict(kind="tensor", n=_log_int(rng, 1000, 100_000_000),
                    mode=rng.choice(("in-hindsight", "in-hindsight", "in-hindsight stochastic", "current", "running")),
                    values=rng.choice(("activation", "gradient")))
    network = rng.choice(("resnet18", "vgg16", "inverted_residual"))
    case = dict(kind="weights", network=network, B=1, image=32 * rng.randint(1, 7))
    if network == "inverted_residual":
        cin = _log_int(rng, 16, 160, 8)
        case.update(cin=cin, cout=_log_int(rng, cin, 160, 8), stride=1)
    return case


# ---------------------------------------------------------------------------------------
# what a training program has in hand before the pass
# ---------------------------------------------------------------------------------------

def _codes(x, scale, zero_point, lo, hi):
    return (x.div_(scale).round_().add_(zero_point).clamp_(lo, hi)).to(torch.int8)


def _activation(g, n, kind):
    """(codes, scale, zero point) of an image (N(0,1), asymmetric), a ReLU6 or a ReLU output."""
    x = torch.randn(n, generator=g, device="cuda")
    if kind == "image":
        lo, hi = float(x.min()), float(x.max())
        scale = (hi - lo) / 255.0
        z = max(-128, min(127, round(-128 - lo / scale)))
        return _codes(x, scale, z, -128, 127), scale, z
    if kind == "relu6":
        return _codes(x.mul_(3.0).clamp_(0.0, 6.0), 6.0 / 255.0, -128, -128, 127), 6.0 / 255.0, -128
    scale = max(float(x.clamp_(min=0.0).max()), 1e-6) / 255.0
    return _codes(x, scale, -128, -128, 127), scale, -128


def _real_gradient(g, n):
    """Laplace(0, 1e-3) with 1 % of the values 20 times as large."""
    u = torch.rand(n, generator=g, device="cuda").sub_(0.5)
    x = u.sign() * torch.log1p(u.abs_().clamp_(max=0.4999999).mul_(-2.0)) * -1e-3
    return torch.where(torch.rand(n, generator=g, device="cuda") < 0.01, x * 20.0, x)


def _gradient(g, n):
    x = _real_gradient(g, n)
    scale = max(float(x.abs().max()), 1e-12) / 127.0
    return _codes(x, scale, 0, -127, 127), scale


class _LayerState:
    """Operands, results and state of one layer."""


def _new_layer(g, L, first, activation):
    s = _LayerState()
    s.L, s.p = L, hq.problem(*L)
    oh, ow = _out_hw(L)
    image = first and L.C == 3
    codes, s.x_scale, s.x_zero = _activation(g, _in_elems(L), "image" if image else activation)
    s.X = codes.view(L.B, L.H, L.W, L.C)
    codes, s.g_scale = _gradient(g, _out_elems(L))
    s.dY = codes.view(L.B, oh, ow, L.Cout)
    s.xq, s.gq = hq.new_qparams(s.x_scale, s.x_zero), hq.new_qparams(s.g_scale, 0)
    s.input_gradient = L.C != 3                                 # a network's first layer has none
    shape = (L.R, L.S, L.C) if L.kind == DEPTHWISE else (L.Cout, L.R, L.S, L.C)
    fan_in = L.R * L.S * (1 if L.kind == DEPTHWISE else L.C)
    real = torch.randn(shape, generator=g, device="cuda") * math.sqrt(2.0 / fan_in)
    s.W, s.wq = torch.empty(shape, dtype=torch.int8, device="cuda"), hq.new_qparams(0, 0)
    hq.hq_weight_quantize(real, real.numel(), s.W, s.wq)
    s.wsum = torch.empty(L.Cout, dtype=torch.int32, device="cuda")
    s.wdsum = torch.empty(L.C, dtype=torch.int32, device="cuda")
    s.Wd = s.W if L.kind == DEPTHWISE else torch.empty((L.C, L.R, L.S, L.Cout), dtype=torch.int8, device="cuda")
    hq.hq_weight_prepare(s.p, s.W, None if L.kind == DEPTHWISE else s.Wd, s.wsum, s.wdsum)
    s.Y = torch.empty_like(s.dY)
    s.dX = torch.empty_like(s.X) if s.input_gradient else None
    s.dW = torch.empty(shape, dtype=torch.float32, device="cuda")
    s.ws_w = hq.hq_workspace_bytes(hq.HQ_ENTRY_WGRAD, s.p)
    s.ws_f = hq.hq_workspace_bytes(hq.HQ_ENTRY_DYNAMIC_FWD, s.p)
    s.ws_d = hq.hq_workspace_bytes(hq.HQ_ENTRY_DYNAMIC_DGRAD, s.p) if s.input_gradient else 0
    return s


def _prepare_layers(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    shapes = _layers(case)
    activation = "relu6" if case["kind"] == "network" and case["network"] == "inverted_residual" else "relu"
    layers = [_new_layer(g, L, i == 0, activation) for i, L in enumerate(shapes)]
    n = len(layers)
    state = {"case": case, "layers": layers, "n": n, "seed": (seed * 0x9E3779B97F4A7C15) % 2 ** 63,
             "ranges": hq.new_ranges([False] * n + [True] * n), "stats": hq.new_stats(2 * n),
             "outq": torch.zeros(2 * n * hq.QPARAMS.itemsize, dtype=torch.uint8, device="cuda")}
    rs, ss, qs = hq.RANGE.itemsize, hq.STATS.itemsize, hq.QPARAMS.itemsize
    for i, s in enumerate(layers):
        s.yr, s.gr = (state["ranges"][k * rs:(k + 1) * rs] for k in (i, n + i))
        s.yst, s.gst = (state["stats"][k * ss:(k + 1) * ss] for k in (i, n + i))
        s.yq, s.dxq = (state["outq"][k * qs:(k + 1) * qs] for k in (i, n + i))
    state["gradient_ranges"], state["gradient_stats"] = state["ranges"][n * rs:], state["stats"][n * ss:]
    # the batch before: its tensors set every range, a little narrower than this batch's
    first = torch.empty(max(max(s.ws_f, s.ws_d) for s in layers), dtype=torch.uint8, device="cuda")
    for s in layers:
        hq.hq_gemm_dynamic(hq.HQ_ENTRY_DYNAMIC_FWD, hq.HQ_DYN_CURRENT, s.p, s.X, hq.new_qparams(0.95 * s.x_scale, s.x_zero),
                           s.W, s.wq, s.wsum, s.yr, s.Y, s.yq, s.yst, first, s.ws_f)
        if s.input_gradient:
            hq.hq_gemm_dynamic(hq.HQ_ENTRY_DYNAMIC_DGRAD, hq.HQ_DYN_CURRENT, s.p, s.dY, hq.new_qparams(0.95 * s.g_scale, 0),
                               s.Wd, s.wq, s.wdsum, s.gr, s.dX, s.dxq, s.gst, first, s.ws_d)
    hq.hq_range_update_batch(state["ranges"], state["stats"], 2 * n)
    # one workspace for the whole stack, of the largest size any of its calls asks for
    dynamic = case.get("ranges", "in-hindsight") != "in-hindsight"
    need = max(max(s.ws_w, s.ws_f if dynamic else 0, s.ws_d if dynamic else 0) for s in layers)
    state["ws"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return state


def _prepare_tensor(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = case["n"]
    x = torch.randn(n, generator=g, device="cuda").clamp_(min=0.0) if case["values"] == "activation" else _real_gradient(g, n)
    state = {"case": case, "x": x, "q": torch.empty(n, dtype=torch.int8, device="cuda"), "seed": (seed * 0x9E3779B97F4A7C15) % 2 ** 63,
             "r": hq.new_range(0.9, case["values"] == "gradient"), "st": hq.new_stats(1), "qp": hq.new_qparams(0, 0)}
    hq.hq_tensor_quantize_dynamic(hq.HQ_DYN_CURRENT, 0.95 * x, n, state["r"], state["q"], state["qp"], state["st"])
    hq.hq_range_update(state["r"], state["st"])
    return state


def _prepare_weights(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    layers, sums = [], 0
    for L in _layers(case):
        s = _LayerState()
        s.L, s.p, s.n = L, hq.problem(*L), _w_elems(L)
        fan_in = L.R * L.S * (1 if L.kind == DEPTHWISE else L.C)
        s.real = torch.randn(s.n, generator=g, device="cuda") * math.sqrt(2.0 / fan_in)
        s.W = torch.empty(s.n, dtype=torch.int8, device="cuda")
        s.Wd = torch.empty(s.n, dtype=torch.int8, device="cuda") if L.kind != DEPTHWISE and L.C != 3 else None
        s.at = sums
        sums += L.Cout + L.C
        layers.append(s)
    state = {"case": case, "layers": layers, "sums": torch.zeros(sums, dtype=torch.int32, device="cuda"),
             "wq": torch.zeros((len(layers), hq.QPARAMS.itemsize), dtype=torch.uint8, device="cuda")}
    for i, s in enumerate(layers):
        s.wq = state["wq"][i]
        s.wsum, s.wdsum = state["sums"][s.at:s.at + s.L.Cout], state["sums"][s.at + s.L.Cout:s.at + s.L.Cout + s.L.C]
    return state


def prepare(case, seed):
    return {"tensor": _prepare_tensor, "weights": _prepare_weights}.get(case["kind"], _prepare_layers)(case, seed)


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------

def _next_seed(state):
    """Stochastic rounding takes another seed for every tensor and iteration."""
    state["seed"] = (state["seed"] + 0x9E3779B97F4A7C15) % 2 ** 64
    return state["seed"]


def _fwd(s):
    hq.hq_gemm_fwd(s.p, s.X, s.xq, s.W, s.wq, s.wsum, s.yr, s.Y, s.yq, s.yst)


def _dgrad(state, s):
    if state["case"]["rounding"] == "stochastic":
        hq.hq_gemm_dgrad_sr(s.p, s.dY, s.gq, s.Wd, s.wq, s.wdsum, s.gr, _next_seed(state), s.dX, s.dxq, s.gst)
    else:
        hq.hq_gemm_dgrad(s.p, s.dY, s.gq, s.Wd, s.wq, s.wdsum, s.gr, s.dX, s.dxq, s.gst)


def _run_layer(state):
    s, ws = state["layers"][0], state["ws"]
    _fwd(s)
    if s.input_gradient:
        _dgrad(state, s)
    hq.hq_gemm_wgrad_update(s.p, s.X, s.xq, s.dY, s.gq, s.dW, None, ws, s.ws_w, state["ranges"], state["stats"], 2)


def _run_layer_dynamic(state):
    s, ws = state["layers"][0], state["ws"]
    mode = hq.HQ_DYN_RUNNING if state["case"]["ranges"] == "running" else hq.HQ_DYN_CURRENT
    hq.hq_gemm_dynamic(hq.HQ_ENTRY_DYNAMIC_FWD, mode, s.p, s.X, s.xq, s.W, s.wq, s.wsum, s.yr, s.Y, s.yq, s.yst, ws, s.ws_f)
    if s.input_gradient and state["case"]["rounding"] == "stochastic":
        hq.hq_gemm_dynamic_sr(hq.HQ_ENTRY_DYNAMIC_DGRAD, mode, s.p, s.dY, s.gq, s.Wd, s.wq, s.wdsum, s.gr, _next_seed(state),
                              s.dX, s.dxq, s.gst, ws, s.ws_d)
    elif s.input_gradient:
        hq.hq_gemm_dynamic(hq.HQ_ENTRY_DYNAMIC_DGRAD, mode, s.p, s.dY, s.gq, s.Wd, s.wq, s.wdsum, s.gr, s.dX, s.dxq, s.gst,
                           ws, s.ws_d)
    hq.hq_gemm_wgrad(s.p, s.X, s.xq, s.dY, s.gq, s.dW, None, ws, s.ws_w)
    hq.hq_stats_reset(state["stats"], 2)


def _run_network(state):
    layers, n, ws = state["layers"], state["n"], state["ws"]
    for s in layers:
        _fwd(s)
    hq.hq_range_update_batch(state["ranges"], state["stats"], n)
    if state["case"]["passes"] == "forward":
        return
    for s in reversed(layers):
        if s.input_gradient:
            _dgrad(state, s)
        hq.hq_gemm_wgrad(s.p, s.X, s.xq, s.dY, s.gq, s.dW, None, ws, s.ws_w)
    hq.hq_range_update_batch(state["gradient_ranges"], state["gradient_stats"], n)


def _run_tensor(state):
    mode, x, n = state["case"]["mode"], state["x"], state["case"]["n"]
    r, q, qp, st = state["r"], state["q"], state["qp"], state["st"]
    if mode == "in-hindsight":
        hq.hq_tensor_quantize(x, n, r, q, qp, st)
    elif mode == "in-hindsight stochastic":
        hq.hq_tensor_quantize_sr(x, n, r, _next_seed(state), q, qp, st)
    else:
        hq.hq_tensor_quantize_dynamic(hq.HQ_DYN_RUNNING if mode == "running" else hq.HQ_DYN_CURRENT, x, n, r, q, qp, st)
        hq.hq_stats_reset(st, 1)
        return {"codes": q, "quantizer": qp, "range": r}
    hq.hq_range_update(r, st)
    return {"codes": q, "quantizer": qp, "range": r}


def _run_weights(state):
    for s in state["layers"]:
        hq.hq_weight_quantize(s.real, s.n, s.W, s.wq)
        hq.hq_weight_prepare(s.p, s.W, s.Wd, s.wsum, s.wdsum)
    return {"codes": [s.W for s in state["layers"]], "relaid": [s.Wd for s in state["layers"]],
            "sums": state["sums"], "quantizers": state["wq"]}


def run(state):
    case = state["case"]
    if case["kind"] == "tensor":
        return _run_tensor(state)
    if case["kind"] == "weights":
        return _run_weights(state)
    if case["kind"] == "network":
        _run_network(state)
    elif case["ranges"] == "in-hindsight":
        _run_layer(state)
    else:
        _run_layer_dynamic(state)
    out = {"Y": [s.Y for s in state["layers"]], "quantizers": state["outq"], "ranges": state["ranges"]}
    if case.get("passes") != "forward":
        out.update(dX=[s.dX for s in state["layers"]], dW=[s.dW for s in state["layers"]])
    return out


# ---------------------------------------------------------------------------------------
# what a pass cannot do without, and how close results have to be
# ---------------------------------------------------------------------------------------

def work(case):
    if case["kind"] == "tensor":
        return {"bytes": 5.0 * case["n"], "flops": 0.0}
    total_bytes, flops = 0.0, 0.0
    for L in _layers(case):
        x, y, w = _in_elems(L), _out_elems(L), _w_elems(L)
        if case["kind"] == "weights":
            total_bytes += 5 * w + (w if L.kind != DEPTHWISE and L.C != 3 else 0) + 4 * (L.C + L.Cout)
        elif case.get("passes") == "forward":
            total_bytes, flops = total_bytes + x + w + y, flops + 2 * _macs(L)
        else:
            # forward X, W -> Y; input gradient dY, W -> dX; weight gradient X, dY -> fp32 dW
            first = L.C == 3
            total_bytes += (x + w + y) + (0 if first else y + w + x) + (x + y + 4 * w)
            flops += 2 * _macs(L) * (2 if first else 3)
    return {"bytes": total_bytes, "flops": flops}


def tolerance(case):
    """Codes, integer sums and statistics are whole numbers, and every fp32 operation behind a code, a range
    or a weight gradient is stated in include/hq.h with its order and rounds once: results are exact."""
    return "exact"
