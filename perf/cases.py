"""Timed cases of the grouped-convolution library, through its public calls.

A case is one of two kinds:
  "conv"  - one gspc_conv2d_grouped call on packed weights (the unit every network is made of);
  "chain" - one gspc_run_layer_chain call, a whole network's forward pass as one recorded graph.
Shapes come from `paper_2006_09791_amd.workloads` (the WRN-40-2-style, ResNet-34-shaped and
MobileNet-shaped networks of the paper's evaluation) or are generic.  Inputs of inner layers are
rectified normal values, what a layer behind a ReLU reads; network inputs are uniform in [-1, 1);
weights are normal with standard deviation sqrt(2 / fan_in).
"""
import math

import torch

from paper_2006_09791_amd import binding
from paper_2006_09791_amd import workloads as wl

DEVICE = "cuda"


def _conv(name, N, Cin, H, W, Cout, k, stride, groups, dtype="f32"):
    return {"name": name, "kind": "conv", "N": N, "Cin": Cin, "H": H, "W": W, "Cout": Cout, "k": k,
            "stride": stride, "pad": k // 2, "groups": groups, "dtype": dtype}


def _chain(name, net, N, groups, pointwise=False):
    return {"name": name, "kind": "chain", "net": net, "N": N, "groups": groups, "pointwise": pointwise}


def listed():
    return [
        # smallest call: one image, one grouped layer; launch and latency decide
        _conv("small_g4", 1, 64, 32, 32, 64, 3, 1, 4),
        # CIFAR-sized residual network at the benchmark's batch: last stage's dense layer, and the
        # stride-2 entry of the second stage in two groups
        _conv("wrn_8x8_g1", 64, 128, 8, 8, 128, 3, 1, 1),
        _conv("wrn_entry_g2", 64, 32, 32, 32, 64, 3, 2, 2),
        # ImageNet-sized residual network, fp32, second stage
        _conv("resnet_28_g2", 64, 128, 28, 28, 128, 3, 1, 2),
        # the same network on bf16 activations at a serving batch: a deep stage where the
        # contraction is wide, and a stage entry where moving the tensors is what there is to do
        _conv("resnet_14_g2_bf16", 256, 256, 14, 14, 256, 3, 1, 2, "bf16"),
        _conv("resnet_56_s2_g8_bf16", 256, 64, 56, 56, 128, 3, 2, 8, "bf16"),
        # depthwise layers of a MobileNet-shaped network: large planes at stride 2, small planes
        _conv("depthwise_112_s2", 256, 64, 112, 112, 64, 3, 2, 64),
        _conv("depthwise_14", 256, 512, 14, 14, 512, 3, 1, 512),
        # the pointwise layer that follows a 3x3 layer in the paper's block form; the largest product
        _conv("pointwise_14", 256, 512, 14, 14, 1024, 1, 1, 1),
        # sizes that fit no tile: odd batch and plane, three groups of 20 channels and 28 filters
        _conv("ragged_g3", 5, 60, 29, 37, 84, 3, 1, 3),
        # whole forward passes: one image (the paper's own measure) and the benchmark's batch
        _chain("resnet34_g4_batch1", "resnet34", 1, 4),
        _chain("wrn_g2_batch64", "wrn", 64, 2),
    ]


# ---- drawn cases -------------------------------------------------------------------------------
MAX_MACS = 40e9         # a drawn layer's multiplications and bytes stay below the largest listed case's
MAX_BYTES = 300e6


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """Per-group channel counts: multiples of 16, of 4 and any number, in turn."""
    v = _log_int(rng, lo, hi)
    m = rng.choice([16, 16, 4, 1])
    return max(lo, (v + m - 1) // m * m)


def draw(rng):
    kind = rng.choice(["conv3", "conv3", "conv3", "bf16", "bf16", "depthwise", "depthwise", "pointwise", "pointwise",
                       "chain"])
    if kind == "chain":
        net = rng.choice(["wrn", "resnet34", "mobilenetv2"])
        pointwise = net != "mobilenetv2" and rng.random() < 0.3
        if net == "wrn":
            case = _chain("", net, _log_int(rng, 1, 64), rng.choice([1, 2, 4, 8, 16]), pointwise)
        elif net == "resnet34":
            case = _chain("", net, _log_int(rng, 1, 8), rng.choice([2, 4, 8, 16, 32]), pointwise)
        else:
            case = _chain("", net, _log_int(rng, 1, 8), rng.choice([2, 4, 8, 16, 0]), False)
    else:
        while True:
            N, H = _log_int(rng, 1, 256), _log_int(rng, 7, 112)
            W = H if rng.random() < 0.7 else _log_int(rng, 7, 112)
            stride = rng.choice([1, 1, 2])
            if kind == "depthwise":
                C = _channels(rng, 16, 1024)
                case = _conv("", N, C, H, W, C, 3, stride, C)
            elif kind == "pointwise":
                case = _conv("", N, _channels(rng, 16, 1024), H, W, _channels(rng, 16, 1024), 1, 1, 1)
            else:
                g = rng.choice([1, 2, 2, 3, 4, 4, 8, 16, 32])
                cpg, kpg = _channels(rng, 2, 128), _channels(rng, 2, 128)
                if rng.random() < 0.6:
                    kpg = cpg
                if g * max(cpg, kpg) > 1024:
                    continue
                case = _conv("", N, g * cpg, H, W, g * kpg, 3, stride, g, "bf16" if kind == "bf16" else "f32")
            w = work(case)
            if w["flops"] <= 2 * MAX_MACS and w["bytes"] <= MAX_BYTES:
                break
    del case["name"]
    return case


# ---- building the state ------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _network(case):
    if case["net"] == "mobilenetv2":
        return wl.mobilenetv2_chain(case["N"], case["groups"] or None)
    build = {"wrn": wl.wrn_chain, "resnet34": wl.resnet34_chain}[case["net"]]
    return build(case["N"], case["groups"], pointwise=case["pointwise"])


def _weight(gen, cout, cpg, kh, kw):
    w = torch.randn((cout, cpg, kh, kw), generator=gen, device=DEVICE)
    return w * math.sqrt(2.0 / (cpg * kh * kw))


def _tensors(case, seed):
    """(input, weights) of a case, from the seed alone."""
    gen = _gen(seed)
    if case["kind"] == "chain":
        ch = _network(case)
        x = torch.rand(ch.input_shape, generator=gen, device=DEVICE) * 2 - 1
        return x, [_weight(gen, *s) for s in ch.weight_shapes]
    x = torch.randn((case["N"], case["Cin"], case["H"], case["W"]), generator=gen, device=DEVICE).clamp_(min=0)
    if case["dtype"] == "bf16":
        x = x.bfloat16()
    return x, [_weight(gen, case["Cout"], case["Cin"] // case["groups"], case["k"], case["k"])]


_side = None     # the stream on which a program runs its recorded chains


def prepare(case, seed):
    global _side
    x, weights = _tensors(case, seed)
    binding.gspc_set_stream()
    if case["kind"] == "conv":
        dtype = binding.GSPC_BF16 if case["dtype"] == "bf16" else binding.GSPC_F32
        pw = binding.gspc_pack_weights(weights[0], case["groups"], dtype)
        ho = wl.out_size(case["H"], case["k"], case["stride"], case["pad"])
        wo = wl.out_size(case["W"], case["k"], case["stride"], case["pad"])
        y = torch.empty((case["N"], case["Cout"], ho, wo), device=DEVICE)
        args = tuple(case[k] for k in ("N", "Cin", "H", "W", "Cout", "k", "k", "stride", "pad", "groups"))
        return {"x": x, "pw": pw, "args": args, "y": y}
    ch = _network(case)
    packed = [binding.gspc_pack_weights(w, g) for w, g in zip(weights, ch.weight_groups)]
    bufs = [torch.empty(max(n, 1), device=DEVICE) for n in ch.buf_elems]
    bufs[0].copy_(x.reshape(-1))
    if _side is None:
        _side = torch.cuda.Stream()
    _side.wait_stream(torch.cuda.current_stream())
    binding.gspc_set_stream(_side)
    out = bufs[ch.out_buf][:math.prod(ch.out_shape)].view(ch.out_shape)
    return {"chain": binding.LayerChain(ch.layers, packed, bufs), "out": out, "stream": _side}


def run(state):
    if "chain" in state:
        binding.gspc_run_layer_chain(state["chain"])
        return state["out"]
    return binding.gspc_conv2d_grouped(state["x"], state["pw"], *state["args"], output=state["y"])


# ---- what a pass cannot do without -------------------------------------------------------------
def work(case):
    if case["kind"] == "chain":
        ch = _network(case)
        elems = math.prod(ch.input_shape) + math.prod(ch.out_shape) + sum(math.prod(s) for s in ch.weight_shapes)
        return {"bytes": 4 * elems, "flops": 2 * ch.macs()}
    s = wl.ConvShape(case["N"], case["Cin"], case["H"], case["W"], case["Cout"], case["k"], case["k"],
                     case["stride"], case["pad"], case["groups"])
    ho, wo = wl.out_size(s.H, s.KH, s.stride, s.pad), wl.out_size(s.W, s.KW, s.stride, s.pad)
    b_in = 2 if case["dtype"] == "bf16" else 4
    wts = s.Cout * (s.Cin // s.groups) * s.KH * s.KW * b_in
    return {"bytes": s.N * s.Cin * s.H * s.W * b_in + wts + s.N * s.Cout * ho * wo * 4,
            "flops": 2 * wl.conv_macs(s)}


def tolerance(case):
    # Products and sums are fp32 everywhere (bf16 layers: exact products of bf16 values, fp32 sums, fp32
    # results).  Measured against exact(): single layers 3e-8 .. 4e-7 (the longest sums and the Winograd
    # layers highest), whole networks 4e-7 .. 8e-7; about four to five times that.
    return {"rel": 4e-6 if case["kind"] == "chain" else 2e-6}


# ---- the same results in 64 bits ---------------------------------------------------------------
def _conv64(x, w, stride, pad, groups):
    """Grouped convolution in float64 by its definition; a few images at a time."""
    N, C, H, W = x.shape
    K, cpg, kh, kw = w.shape
    ho, wo = wl.out_size(H, kh, stride, pad), wl.out_size(W, kw, stride, pad)
    y = torch.empty((N, K, ho, wo), dtype=torch.float64, device=x.device)
    step = max(1, int(5e8 // (8 * C * kh * kw * ho * wo)))
    for n in range(0, N, step):
        xp = torch.nn.functional.pad(x[n:n + step], (pad, pad, pad, pad))
        m = xp.shape[0]

        def window(i, j):
            return xp[:, :, i:i + stride * (ho - 1) + 1:stride, j:j + stride * (wo - 1) + 1:stride]

        if cpg == 1 and K == C:
            y[n:n + m] = sum(window(i, j) * w[:, 0, i, j].view(1, C, 1, 1) for i in range(kh) for j in range(kw))
            continue
        cols = torch.stack([window(i, j) for i in range(kh) for j in range(kw)], 2)
        cols = cols.reshape(m, groups, cpg * kh * kw, ho * wo)
        wg = w.reshape(1, groups, K // groups, cpg * kh * kw)
        y[n:n + m] = torch.matmul(wg, cols).reshape(m, K, ho, wo)
    return y


def exact(case, seed):
    x, weights = _tensors(case, seed)
    if case["kind"] == "conv":
        w = weights[0].bfloat16() if case["dtype"] == "bf16" else weights[0]
        return _conv64(x.double(), w.double(), case["stride"], case["pad"], case["groups"])
    ch = _network(case)
    bufs = {0: x.double()}
    for l in ch.layers:
        if l.op == "maxpool":
            bufs[l.dst] = torch.nn.functional.max_pool2d(bufs[l.src], l.KH, l.stride, l.pad)
            continue
        y = _conv64(bufs[l.src], weights[l.wid].double(), l.stride, l.pad, l.groups)
        if l.src2 >= 0:
            y = y + bufs[l.src2]
        bufs[l.dst] = y.clamp(min=0) if l.relu else y
    return bufs[ch.out_buf]
