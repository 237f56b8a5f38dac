"""Performance cases of the quantized-layer library: what a program built on it asks of it, from the smallest call to a
whole stage of a U-Net.

A case is a dict of plain values.  `kind` names the piece of work:

  linear    one linear layer: fp32 activations (dynamic or calibrated scale) or codes in, fp32 out
  conv      one convolution, the same options; odd sizes, widths and formats included
  ff        a transformer feed-forward block with calibrated scales: the projection hands its gated result to the second
            layer as codes
  group     the key / value projections of several cross-attention blocks in one grouped call
  stage     every conv / linear layer of one U-Net stage (a ResNet block and a transformer block), scales found per layer
  search    encoding and bias search (Algorithm 1 of the paper) over one activation tensor
  rounding  one gradient step of rounding learning on one layer's weights
  sparse    one convolution on the structured-sparse weight operand
  integer   the integer baseline on one linear layer: calibrate, quantize, multiply

Weights are quantized and packed in prepare(), as a program does once when it loads a model.
"""
import math

import torch

from paper_2408_06995_amd import binding as fpq
from paper_2408_06995_amd import synth

DEVICE = "cuda:0"
FORMATS = {"e4m3": synth.E4M3, "e2m1": synth.E2M1, "e3m4": synth.E3M4, "e3m0": synth.E3M0}
SEARCH_ENCODINGS = {8: [(2, 5), (3, 4), (4, 3), (5, 2)], 4: [(2, 1), (1, 2)]}   # candidates for eight and for four bits
SEARCH_BIASES = 111                                                             # bias candidates per encoding, as in the paper


# ------------------------------------------------------------------------------------------------ the cases

def listed():
    return [
        # A time-embedding projection at batch 8: the smallest layer of a U-Net step, 22 of them per step.
        dict(name="time_embedding", kind="linear", M=8, K=1280, N=1280, x="dynamic", w="e4m3", acc="fp32", bias=True),
        # Key / value projections of the cross-attention blocks at batch 8 (77 text tokens of width 768): independent of
        # the layers between them, so a program makes them one call.
        dict(name="context_kv", kind="group", count=32, M=616, K=768, N=320, w="e2m1"),
        # The query / key / value projection of the finest level at batch 4, activations already codes: compute through
        # the 8-bit matrix instruction, the option for callers that accept its tolerance.
        dict(name="qkv_fp8_mfma", kind="linear", M=16384, K=320, N=960, x="codes", w="e4m3", acc="fp8", bias=True),
        # Feed-forward block of the finest level at batch 4, scales calibrated offline as in the paper.
        dict(name="feed_forward", kind="ff", M=16384, C=320, w="e4m3"),
        # 3x3 convolution of the finest level at batch 1: one image, latency.
        dict(name="conv_320_64_b1", kind="conv", B=1, C=320, H=64, W=64, N=320, k=3, stride=1, x="dynamic", f="e4m3", w="e4m3"),
        # Deep-stage convolution with 4-bit weights at batch 8: the paper's headline setting.
        dict(name="conv_1280_16_w4", kind="conv", B=8, C=1280, H=16, W=16, N=1280, k=3, stride=1, x="dynamic", f="e4m3", w="e2m1"),
        # The same stage in encodings the hardware has no instruction for, as the format sweep uses them.
        dict(name="conv_1280_16_e3m4_e3m0", kind="conv", B=8, C=1280, H=16, W=16, N=1280, k=3, stride=1, x="static", f="e3m4",
             w="e3m0"),
        # A picture that is no power of two through a network of other widths, batch 3, strided.
        dict(name="conv_ragged", kind="conv", B=3, C=200, H=75, W=53, N=392, k=3, stride=2, x="dynamic", f="e4m3", w="e4m3"),
        # The first decoder stage of the finest level: 640 concatenated channels to 320 at batch 8.
        dict(name="stage_320_64", kind="stage", B=8, Cin=640, C=320, R=64, w="e4m3"),
        # Calibration, per activation tensor: four encodings x 111 biases on a finest-level activation.
        dict(name="search_320_64", kind="search", n=8 * 320 * 64 * 64, bits=8),
        # Rounding learning, per layer and iteration: a 1280 x 1280 projection on 8192 calibration rows.
        dict(name="rounding_1280", kind="rounding", M=8192, N=1280, K=1280, w="e2m1"),
        # The paper's comparison system, integers of the same width, on the widest projection it would replace.  (Pruned
        # weights, the other alternative operand, are among the drawn cases.)
        dict(name="integer_1280_10240", kind="integer", M=2048, K=1280, N=10240, bits=8),
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _step(v, s):
    return max(s, v // s * s)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "conv", "conv", "conv", "ff", "group", "stage", "search", "rounding",
                       "sparse", "integer"])
    w = rng.choice(["e4m3", "e2m1"])
    if kind == "linear":
        while True:
            c = dict(kind=kind, M=_log(rng, 1, 32768), K=_log(rng, 64, 5120), N=_log(rng, 16, 10240),
                     x=rng.choice(["dynamic", "static", "codes"]), w=w, acc=rng.choice(["fp32", "fp32", "fp8"]),
                     bias=rng.random() < 0.5)
            if rng.random() < 0.5:                       # network widths are multiples of 64 as a rule
                c["K"], c["N"] = _step(c["K"], 64), _step(c["N"], 64)
            if c["x"] == "codes":
                c["K"] = _step(c["K"], 16)               # what code operands ask for
            if c["M"] * c["K"] * c["N"] <= 32768 * 320 * 2560:
                return c
    if kind == "conv":
        while True:
            f = rng.choice(["e4m3", "e4m3", "e4m3", "e3m4"])
            c = dict(kind=kind, B=_log(rng, 1, 8), C=_log(rng, 4, 1920), H=_log(rng, 8, 96), W=_log(rng, 8, 96),
                     N=_log(rng, 4, 1280), k=rng.choice([3, 3, 1]), stride=rng.choice([1, 1, 1, 2]),
                     x=rng.choice(["dynamic", "static", "codes"]), f=f, w="e3m0" if f == "e3m4" else w)
            if rng.random() < 0.5:
                c["C"], c["N"] = _step(c["C"], 32), _step(c["N"], 32)
            if _conv_flops(c) <= 2 * 8192 * 11520 * 640:
                return c
    if kind == "ff":
        while True:
            c = dict(kind=kind, M=_log(rng, 64, 32768), C=_step(_log(rng, 64, 1280), 32), w=w)
            if c["M"] * c["C"] ** 2 <= 16384 * 320 ** 2 * 2:
                return c
    if kind == "group":
        return dict(kind=kind, count=rng.randint(4, 40), M=_log(rng, 8, 1024), K=_step(_log(rng, 128, 1280), 16),
                    N=_step(_log(rng, 64, 640), 16), w=w)
    if kind == "stage":
        while True:
            C = _step(_log(rng, 128, 1280), 32)
            c = dict(kind=kind, B=rng.randint(1, 8), Cin=rng.choice([C, 2 * C, _step(C + C // 2, 32)]), C=C, R=_log(rng, 8, 64), w=w)
            if c["B"] * c["R"] ** 2 * (9 * c["Cin"] + 9 * C + 22 * C) * C <= 8 * 64 ** 2 * (9 * 640 + 31 * 320) * 320:
                return c
    if kind == "search":
        return dict(kind=kind, n=_log(rng, 10000, 8 * 320 * 64 * 64), bits=rng.choice([8, 8, 4]))
    if kind == "rounding":
        while True:
            c = dict(kind=kind, M=_log(rng, 256, 16384), N=_log(rng, 64, 1280), K=_log(rng, 64, 2880), w=w)
            if c["M"] * c["N"] * c["K"] <= 8192 * 1280 * 1280:
                return c
    if kind == "sparse":
        while True:
            c = dict(kind=kind, B=_log(rng, 1, 8), C=_log(rng, 32, 1280), H=_log(rng, 8, 64), W=_log(rng, 8, 64),
                     N=_log(rng, 32, 1280), k=rng.choice([3, 3, 1]), stride=1, w=w)
            if _conv_flops(c) <= 2 * 2048 * 11520 * 1280:
                return c
    while True:
        c = dict(kind=kind, M=_log(rng, 16, 32768), K=_step(_log(rng, 64, 5120), 16), N=_log(rng, 64, 10240),
                 bits=rng.choice([8, 4]))
        if c["M"] * c["K"] * c["N"] <= 32768 * 320 * 2560:
            return c


# ------------------------------------------------------------------------------------------------ inputs

def _u8(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEVICE)


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEVICE)


def _seed(seed, i):
    return seed * 1000 + i


def _static_scale(x, f):
    """The calibrated per-tensor scale absmax / max value, as a host number."""
    n = x.numel()
    ws, out = _f32(max(2, fpq.fpq_absmax_workspace_size(n) // 4)), _f32(2)
    fpq.fpq_absmax(x, f[3], out[0:1], out[1:2], ws)
    return float(out[1].item())


def _pack(w, f, mask):
    N, C = w.shape[:2]
    kh, kw = (w.shape[2], w.shape[3]) if w.dim() == 4 else (1, 1)
    packed, sw = _u8(fpq.fpq_packed_size(N, C, kh, kw, f)), _f32(N)
    fpq.fpq_pack_weights(w, f, None, mask, packed, sw)
    return packed, sw


def _layer_weights(shape, f, seed, bias=False):
    """Packed weights with a random rounding mask, their scales, and a bias or None."""
    w = synth.weights_torch(shape, seed + 500, DEVICE)
    packed, sw = _pack(w, f, synth.rounding_mask_torch(shape, seed + 750, DEVICE))
    b = None
    if bias:
        g = torch.Generator(device=DEVICE)
        g.manual_seed(seed + 900)
        b = torch.randn(shape[0], generator=g, device=DEVICE) * 0.1
    return packed, sw, b


X_KIND = {"codes": fpq.FPQ_X_CODES, "static": fpq.FPQ_X_FP32, "dynamic": fpq.FPQ_X_FP32_DYNAMIC}


def _linear(M, K, N, x_form, wf, seed, acc="fp32", bias=False):
    """Arguments of one fpq_gemm call."""
    fx, fw = synth.E4M3, FORMATS[wf]
    x = synth.activations_torch((M, K), seed, DEVICE)
    sx = 0.0 if x_form == "dynamic" else _static_scale(x, fx)
    if x_form == "codes":
        codes = _u8(M * K)
        fpq.fpq_quantize(x, fx, sx, None, codes)
        x = codes
    packed, sw, b = _layer_weights((N, K), fw, seed, bias)
    kind = X_KIND[x_form]
    ws = _u8(fpq.fpq_gemm_workspace_size(M, N, K, kind))
    mode = fpq.FPQ_ACC_FP8_MFMA if acc == "fp8" else fpq.FPQ_ACC_FP32
    return (x, kind, fx, sx, None, packed, fw, sw, b, _f32(M, N), M, N, K, mode, ws)


def _out(c):
    pad = c["k"] // 2
    return pad, (c["H"] + 2 * pad - c["k"]) // c["stride"] + 1, (c["W"] + 2 * pad - c["k"]) // c["stride"] + 1


def _conv_flops(c):
    _, ho, wo = _out(c)
    return 2 * c["B"] * ho * wo * c["C"] * c["k"] ** 2 * c["N"]


def _conv(c, seed, x_form, sparse=False):
    """Arguments of one fpq_conv2d (or fpq_conv2d_sparse) call."""
    fx, fw = FORMATS[c.get("f", "e4m3")], FORMATS[c["w"]]
    B, C, H, W, N, k, stride = (c[v] for v in ("B", "C", "H", "W", "N", "k", "stride"))
    pad, ho, wo = _out(c)
    x = synth.activations_torch((B, C, H, W), seed, DEVICE)
    sx = 0.0 if x_form == "dynamic" else _static_scale(x, fx)
    if x_form == "codes":
        codes = _u8(B * H * W * fpq.fpq_padded_channels(C))
        fpq.fpq_quantize_nhwc(x, fx, sx, None, codes)
        x = codes
    kind = X_KIND[x_form]
    ws = _u8(fpq.fpq_conv2d_workspace_size(B, C, H, W, N, k, k, stride, pad, kind))
    y = _f32(B, N, ho, wo)
    if sparse:
        w = synth.weights_torch((N, C, k, k), seed + 500, DEVICE)
        packed, sw = _u8(fpq.fpq_packed_sparse_size(N, C, k, k, fw)), _f32(N)
        dropped = torch.zeros(1, dtype=torch.int64, device=DEVICE)
        fpq.fpq_pack_weights_sparse(w, fw, None, synth.rounding_mask_torch(tuple(w.shape), seed + 750, DEVICE), packed, sw, None,
                                    dropped)
        return (x, kind, fx, sx, None, packed, fw, sw, None, y, B, C, H, W, N, k, k, stride, pad, ws)
    packed, sw, b = _layer_weights((N, C, k, k), fw, seed, bias=True)
    return (x, kind, fx, sx, None, packed, fw, sw, b, y, B, C, H, W, N, k, k, stride, pad, fpq.FPQ_ACC_FP32, ws)


def _stage_layers(c):
    """The layers of one stage: (name, what, sizes).  A ResNet block, then a transformer block."""
    B, C, R = c["B"], c["C"], c["R"]
    M = B * R * R

    def conv(name, ci, k):
        return (name, "conv", dict(B=B, C=ci, H=R, W=R, N=C, k=k, stride=1, w=c["w"]))

    def lin(name, m, k, n):
        return (name, "linear", dict(M=m, K=k, N=n))

    layers = [conv("conv1", c["Cin"], 3), lin("temb", B, 1280, C), conv("conv2", C, 3)]
    if c["Cin"] != C:
        layers.append(conv("skip", c["Cin"], 1))
    layers += [conv("proj_in", C, 1), lin("attn1_qkv", M, C, 3 * C), lin("attn1_out", M, C, C), lin("attn2_q", M, C, C),
               ("attn2_kv", "group", dict(count=2, M=B * 77, K=768, N=C)), lin("attn2_out", M, C, C),
               lin("ff_geglu", M, C, 8 * C), lin("ff_out", M, 4 * C, C), conv("proj_out", C, 1)]
    return layers


def _group(count, M, K, widths, wf, seed):
    fw = FORMATS[wf]
    items, keep, ys = [], [], []
    for i in range(count):
        x = synth.activations_torch((M, K), _seed(seed, i), DEVICE)
        packed, sw, _ = _layer_weights((widths[i], K), fw, _seed(seed, i))
        y = _f32(M, widths[i])
        items.append((x, None, packed, sw, None, y, M, widths[i], K))
        keep.append((x, packed, sw))
        ys.append(y)
    problems = fpq.gemm_problems(items)
    ws = _u8(fpq.fpq_gemm_grouped_workspace_size(problems, fpq.FPQ_X_FP32_DYNAMIC))
    return {"args": (problems, fpq.FPQ_X_FP32_DYNAMIC, synth.E4M3, fw, fpq.FPQ_ACC_FP32, ws), "y": ys, "keep": keep}


def _group_widths(c):
    """Blocks of a U-Net's levels: the base width, twice and four times that, a pair (key, value) each."""
    return [c["N"] * (1, 1, 2, 2, 4, 4)[i % 6] for i in range(c["count"])]


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"kind": kind}
    if kind == "linear":
        s["args"] = _linear(c["M"], c["K"], c["N"], c["x"], c["w"], seed, c["acc"], c["bias"])
    elif kind == "conv":
        s["args"] = _conv(c, seed, c["x"])
    elif kind == "sparse":
        s["args"] = _conv(c, seed, "dynamic", sparse=True)
    elif kind == "group":
        s["group"] = _group(c["count"], c["M"], c["K"], _group_widths(c), c["w"], seed)
    elif kind == "ff":
        M, C = c["M"], c["C"]
        x, xk, fx, sx, _, p1, fw, sw1, b1, _, _, _, _, mode, _ = _linear(M, C, 8 * C, "static", c["w"], seed, bias=True)
        p2, sw2, b2 = _layer_weights((C, 4 * C), fw, seed + 1, bias=True)
        # clip of the hidden activations: six standard deviations of value and gate, as a calibration run would set it
        sy = 36.0 * (0.025 ** 2 * C) / synth.E4M3[3]
        hidden = torch.empty((M, 4 * C), dtype=torch.uint8, device=DEVICE)
        ws1 = _u8(fpq.fpq_gemm_workspace_size(M, 8 * C, C, xk))
        ws2 = _u8(fpq.fpq_gemm_workspace_size(M, C, 4 * C, fpq.FPQ_X_CODES))
        s["first"] = (x, xk, fx, sx, None, p1, fw, sw1, b1, fx, sy, None, hidden, M, 8 * C, C, fpq.FPQ_ACC_FP32 | fpq.FPQ_ACT_GEGLU,
                      ws1)
        s["second"] = (hidden, fpq.FPQ_X_CODES, fx, sy, None, p2, fw, sw2, b2, _f32(M, C), M, C, 4 * C, fpq.FPQ_ACC_FP32, ws2)
    elif kind == "stage":
        s["layers"] = []
        for i, (name, what, z) in enumerate(_stage_layers(c)):
            at = _seed(seed, i)
            if what == "conv":
                s["layers"].append((name, what, _conv(z, at, "dynamic")))
            elif what == "linear":
                s["layers"].append((name, what, _linear(z["M"], z["K"], z["N"], "dynamic", c["w"], at, bias=True)))
            else:
                s["layers"].append((name, what, _group(z["count"], z["M"], z["K"], [z["N"]] * z["count"], c["w"], at)))
    elif kind == "search":
        x = synth.activations_torch((c["n"],), seed, DEVICE)
        encodings = SEARCH_ENCODINGS[c["bits"]]
        ne = len(encodings)
        ws = _u8(fpq.fpq_search_workspace_size(c["n"], ne, SEARCH_BIASES))
        s["args"] = (x, encodings, SEARCH_BIASES, _f32(ne * SEARCH_BIASES), _u8(256), ws)
    elif kind == "rounding":
        M, N, K, f = c["M"], c["N"], c["K"], FORMATS[c["w"]]
        w = synth.weights_torch((N, K), seed + 500, DEVICE)
        _, sw = _pack(w, f, None)
        alpha = torch.empty_like(w)
        fpq.fpq_rl_init_alpha(w, sw, f, alpha)
        a = synth.activations_torch((M, K), seed, DEVICE)
        ws = _u8(fpq.fpq_rl_workspace_size(M, N, K))
        s["args"] = (w, sw, f, alpha, a, 1e-2, 1e-3, _f32(2), _f32(N, K), ws)
    else:   # integer
        M, K, N = c["M"], c["K"], c["N"]
        x = synth.activations_torch((M, K), seed, DEVICE)
        w = synth.weights_torch((N, K), seed + 500, DEVICE)
        packed, sw = _u8(fpq.fpq_int_packed_size(N, K, c["bits"])), _f32(N)
        zw = torch.empty(N, dtype=torch.int32, device=DEVICE)
        fpq.fpq_int_pack_weights(w, c["bits"], packed, sw, zw)
        codes = torch.empty((M, K), dtype=torch.uint8, device=DEVICE)
        params = torch.empty(16, dtype=torch.uint8, device=DEVICE)
        s["calibrate"] = (x, 8, params, _u8(fpq.lib().fpq_int_calibrate_workspace_size(x.numel())))
        s["quantize"] = (x, 8, 1.0, 0, params, codes)
        s["args"] = (codes, 1.0, 0, params, packed, c["bits"], sw, zw, None, _f32(M, N), M, N, K,
                     _u8(fpq.fpq_int_gemm_workspace_size(M)))
    return s


# ------------------------------------------------------------------------------------------------ one pass

def run(state):
    kind = state["kind"]
    if kind == "linear":
        fpq.fpq_gemm(*state["args"])
        return state["args"][9]
    if kind == "conv":
        fpq.fpq_conv2d(*state["args"])
        return state["args"][9]
    if kind == "sparse":
        fpq.fpq_conv2d_sparse(*state["args"])
        return state["args"][9]
    if kind == "group":
        fpq.fpq_gemm_grouped(*state["group"]["args"])
        return state["group"]["y"]
    if kind == "ff":
        fpq.fpq_gemm_codes_out(*state["first"])
        fpq.fpq_gemm(*state["second"])
        return {"hidden": state["first"][12], "y": state["second"][9]}
    if kind == "stage":
        out = {}
        for name, what, args in state["layers"]:
            if what == "conv":
                fpq.fpq_conv2d(*args)
                out[name] = args[9]
            elif what == "linear":
                fpq.fpq_gemm(*args)
                out[name] = args[9]
            else:
                fpq.fpq_gemm_grouped(*args["args"])
                out[name] = args["y"]
        return out
    if kind == "search":
        fpq.fpq_search_format(*state["args"])
        mse, result = state["args"][3], state["args"][4]
        return {"mse": mse, "chosen": result[:20].view(torch.int32), "values": result[20:36].view(torch.float32)}
    if kind == "rounding":
        fpq.fpq_rl_step(*state["args"])
        return {"alpha": state["args"][3], "loss": state["args"][7], "grad": state["args"][8]}
    fpq.fpq_int_calibrate(*state["calibrate"])
    fpq.fpq_int_quantize(*state["quantize"])
    fpq.fpq_int_gemm(*state["args"])
    return {"codes": state["quantize"][5], "y": state["args"][9]}


# ------------------------------------------------------------------------------------------------ what a pass needs

def _weight_bytes(wf, n):
    e, m = FORMATS[wf][:2]
    return n / 2 if 1 + e + m <= 4 else n


def _sum(parts):
    return {"bytes": float(sum(p["bytes"] for p in parts)), "flops": float(sum(p["flops"] for p in parts))}


def _linear_work(M, K, N, x, w):
    return {"bytes": M * K * (1 if x == "codes" else 4) + _weight_bytes(w, N * K) + 4 * M * N, "flops": 2 * M * K * N}


def _conv_work(c, x, sparse=False):
    _, ho, wo = _out(c)
    wb = _weight_bytes(c["w"], c["N"] * c["C"] * c["k"] ** 2)
    if sparse:                                            # half the codes and two position bits for each of them
        wb = wb / 2 + c["N"] * c["C"] * c["k"] ** 2 / 8
    return {"bytes": c["B"] * c["C"] * c["H"] * c["W"] * (1 if x == "codes" else 4) + wb + 4 * c["B"] * c["N"] * ho * wo,
            "flops": _conv_flops(c) / (2 if sparse else 1)}


def work(case):
    c, kind = case, case["kind"]
    if kind == "linear":
        return _sum([_linear_work(c["M"], c["K"], c["N"], c["x"], c["w"])])
    if kind == "conv":
        return _sum([_conv_work(c, c["x"])])
    if kind == "sparse":
        return _sum([_conv_work(c, "dynamic", sparse=True)])
    if kind == "group":
        return _sum([_linear_work(c["M"], c["K"], n, "dynamic", c["w"]) for n in _group_widths(c)])
    if kind == "ff":
        M, C = c["M"], c["C"]
        return {"bytes": float(4 * M * C + _weight_bytes(c["w"], 12 * C * C) + 4 * M * C + 4 * M * C), "flops": float(24 * M * C * C)}
    if kind == "stage":
        parts = []
        for _, what, z in _stage_layers(c):
            if what == "conv":
                parts.append(_conv_work(z, "dynamic"))
            else:
                parts += [_linear_work(z["M"], z["K"], z["N"], "dynamic", c["w"])] * z.get("count", 1)
        return _sum(parts)
    if kind == "search":
        # a squared difference per element, at least one read of the tensor; the candidates can share what they have in common
        return {"bytes": 4.0 * c["n"], "flops": 3.0 * c["n"]}
    if kind == "rounding":
        M, N, K = c["M"], c["N"], c["K"]
        return {"bytes": 4.0 * (M * K + 4 * N * K), "flops": 4.0 * M * N * K}
    M, K, N = c["M"], c["K"], c["N"]
    return {"bytes": float(5 * M * K + N * K * c["bits"] // 8 + 4 * M * N), "flops": float(2 * M * K * N)}


def tolerance(case):
    kind = case["kind"]
    if kind == "linear" and case["acc"] == "fp8":
        return {"rel": 1e-3}                              # the 8-bit instruction drops bits 2^-13 below a group's largest product
    if kind == "ff":
        # a hidden value that lies on a rounding boundary within the 32-bit sums' own error takes either code
        return {"rel": 1e-3, "max": 0.1, "differ": 1e-3}
    if kind == "integer":
        return {"rel": 1e-6}                              # exact integer sums, one 32-bit scaling
    if kind == "rounding":
        return {"rel": 2e-5, "max": 1e-3}                 # two 32-bit products in a row
    return {"rel": 1e-5}                                  # 32-bit sums of exact products; errors of the search likewise
