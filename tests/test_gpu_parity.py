"""GPU parity: the HIP path (through the C ABI) against the CPU oracle on the same seeded inputs.
Codes must match bit for bit; layer outputs must satisfy |gpu - oracle| <= 1e-5 * sum_k|a_k b_k| + 1e-6
in the fp32-accumulate mode (the default), and the hardware bound 7 * 2^-13 * sum_k|a_k b_k| in the
FP8-MFMA mode, whose matrix unit drops product bits more than 13 places below the largest of each 8."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, check_close, dev, gpu_absmax_scale, gpu_pack, gpu_quantize, oracle_linear_inputs

pytestmark = pytest.mark.gpu

FORMATS = {
    "E4M3": synth.E4M3, "E5M2": synth.E5M2, "E2M1": synth.E2M1, "E1M2": synth.E1M2, "E3M4": synth.E3M4,
    "E2M5": synth.E2M5, "E3M0": synth.E3M0, "E4M3_eq7": (4, 3, 7, 480.0), "E4M3_b9": (4, 3, 9, 112.0),
    "E5M2_eq7": (5, 2, 15, 0.0), "E2M1_b2": (2, 1, 2, 3.0), "E3M2": (3, 2, 3, 28.0), "E1M6": (1, 6, 1, 0.0),
    "E4M3_bneg": (4, 3, -3, 0.0), "E2M3_sub": (2, 3, 1, 0.875),
}
REL_FP8_MFMA = 7 * 2.0 ** -13


def resolved(f):
    e, m, b, c = f
    return (e, m, b, c if c else oracle.format_max(e, m, b))


def edge_values(f, scale):
    e, m, b, c = resolved(f)
    g = oracle.grid((e, m, b, c))
    g = g[g <= c]
    mids = (g[:-1] + g[1:]) / 2
    v = np.concatenate([g, mids, [c * 1.01, c * 4, 0.0]]).astype(np.float32)
    v = np.concatenate([v, np.nextafter(v, np.float32(np.inf)), np.nextafter(v, np.float32(-np.inf))])
    v = np.concatenate([v, -v, np.array([np.inf, -np.inf, -0.0, 1e-45, -1e-45, 1e-38, 3e38], dtype=np.float32)])
    return (v.astype(np.float64) * float(scale)).astype(np.float32)


# ------------------------------------------------------------------------------ quantizer

@pytest.mark.parametrize("name", sorted(FORMATS))
def test_quantize_codes_bit_exact(name):
    f = resolved(FORMATS[name])
    rng = np.random.default_rng(abs(hash(name)) % 2 ** 31)
    four = 1 + f[0] + f[1] <= 4
    for scale in (1.0, 0.0371, 2.0 ** -4, 5.3):
        scale = float(np.float32(scale))
        x = np.concatenate([synth.activations((70001,), 11) * np.float32(scale * f[3] / 4),
                            rng.uniform(-1.5, 1.5, 30000).astype(np.float32) * np.float32(scale * f[3]),
                            edge_values(f, scale), edge_values(f, 1.0)])
        want = oracle.quantize(x, f, scale)
        got = gpu_quantize(x, f, scale)
        if four:
            want = oracle.pack4(want)
        assert got.shape == want.shape
        assert np.array_equal(got, want), "%s scale %g: %d codes differ" % (name, scale, int((got != want).sum()))
    # device-resident scale gives the same codes
    x = synth.activations((4099,), 12)
    sd = dev(np.array([0.0371], dtype=np.float32))
    got = gpu_quantize(x, f, None, sd)
    want = oracle.quantize(x, f, float(np.float32(0.0371)))
    assert np.array_equal(got, oracle.pack4(want) if four else want)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 63, 255, 1023, 4097, 262147])
def test_quantize_ragged_sizes_and_alignment(n):
    for f in (synth.E4M3, synth.E2M1):
        x = synth.activations((n + 3,), 100 + n)
        for off in (0, 1):                       # off = 1: 4-byte-aligned but not 16-byte-aligned input
            xs = x[off:off + n]
            xt = dev(x)[off:off + n]
            codes = torch.full((B.fpq_code_bytes(n, f) + 8,), 0xEE, dtype=torch.uint8, device=DEV)
            B.fpq_quantize(xt, f, 0.02, None, codes[4:])
            torch.cuda.synchronize()
            got = codes.cpu().numpy()
            want = oracle.quantize(xs, f, float(np.float32(0.02)))
            if f is synth.E2M1:
                want = oracle.pack4(want)
            assert np.array_equal(got[4:4 + want.size], want)
            assert np.all(got[:4] == 0xEE) and np.all(got[4 + want.size:] == 0xEE)   # nothing written outside


def test_quantize_strided_sweep_of_all_fp32_patterns():
    """Every 257th fp32 bit pattern (16.7 M inputs: all exponents, denormals, both signs, infinities)."""
    bits = np.arange(0, 2 ** 32, 257, dtype=np.uint64).astype(np.uint32)
    x = bits.view(np.float32)
    x = x[~np.isnan(x)]
    for f, scale in ((synth.E4M3, 1.0), (synth.E4M3, 0.7331), (synth.E3M4, 1.0), (synth.E2M1, 3.0e-3), (synth.E5M2, 1e-30)):
        scale = float(np.float32(scale))
        want = oracle.quantize(x, f, scale)
        if 1 + f[0] + f[1] <= 4:
            want = oracle.pack4(want)
        got = gpu_quantize(x, f, scale)
        assert np.array_equal(got, want), (f, scale, int((got != want).sum()))


def test_absmax_and_scale():
    for n in (1, 5, 4096, 4097, 1310720, 5000001):
        x = synth.activations((n,), 7 + n)
        out = gpu_absmax_scale(dev(x), 448.0).cpu().numpy()
        a = oracle.absmax(x)
        assert out[0] == np.float32(a)
        assert out[1] == np.float32(oracle.scale_from_absmax(a, 448.0))
    z = gpu_absmax_scale(torch.zeros(1000, device=DEV), 448.0).cpu().numpy()
    assert z[0] == 0.0 and z[1] == 1.0
    e = gpu_absmax_scale(torch.zeros(0, device=DEV), 6.0).cpu().numpy()
    assert e[0] == 0.0 and e[1] == 1.0
    x = synth.activations((1001,), 3)
    out = gpu_absmax_scale(dev(x)[1:], 6.0).cpu().numpy()       # unaligned start
    assert out[0] == np.float32(oracle.absmax(x[1:]))


@pytest.mark.parametrize("shape", [(1, 320, 64, 64), (2, 4, 9, 7), (3, 20, 5, 5), (1, 70, 1, 1), (2, 130, 16, 16)])
def test_quantize_nhwc(shape):
    f = synth.E4M3
    x = synth.activations(shape, 41)
    sx = oracle.scale_from_absmax(oracle.absmax(x), f[3])
    Bn, Cc, H, W = shape
    Cp = B.fpq_padded_channels(Cc)
    codes = torch.full((Bn * H * W * Cp,), 0xEE, dtype=torch.uint8, device=DEV)
    B.fpq_quantize_nhwc(dev(x), f, sx, None, codes)
    torch.cuda.synchronize()
    got = codes.cpu().numpy().reshape(Bn, H, W, Cp)
    want = oracle.quantize(x, f, sx).transpose(0, 2, 3, 1)
    assert np.array_equal(got[..., :Cc], want)
    assert np.all(got[..., Cc:] == 0)


# ------------------------------------------------------------------------------ weights

@pytest.mark.parametrize("name", ["E2M1", "E4M3", "E1M2", "E3M0", "E3M4", "E2M1_b2", "E5M2"])
@pytest.mark.parametrize("shape", [(320, 320), (7, 40, 3, 3), (33, 5, 1, 1), (4, 320, 3, 3)])
def test_pack_weights_codes_and_scales(name, shape):
    f = resolved(FORMATS[name])
    w = synth.weights(shape, 4500)
    w.reshape(-1)[::97] = 0.0
    h = synth.rounding_mask(shape, 4750)
    for mask in (h, None):
        want_codes, want_sw = oracle.pack_weights(w, f, mask)
        _, sw, codes = gpu_pack(w, f, mask)
        assert np.array_equal(sw.cpu().numpy(), want_sw)
        assert np.array_equal(codes, want_codes), int((codes != want_codes).sum())
    # given scales, and on-grid / clipped weights under the mask (Eq. (12) literally)
    sc = np.full(shape[0], 0.013, dtype=np.float32)
    g = oracle.grid(f)
    wg = (np.resize(np.concatenate([g, -g, [2 * f[3], -2 * f[3]]]), w.size).reshape(shape) * 0.013).astype(np.float32)
    want_codes, _ = oracle.pack_weights(wg, f, h, sc)
    _, sw, codes = gpu_pack(wg, f, h, sc)
    assert np.array_equal(codes, want_codes) and np.array_equal(sw.cpu().numpy(), sc)


# ------------------------------------------------------------------------------ linear layers

def run_linear(x, w, h, fx, fw, acc, bias=None, fp32_in=False):
    sx, xq, wq, sw = oracle_linear_inputs(x, w, h, fx, fw)
    M, K = x.shape
    N = w.shape[0]
    packed, sw_t, codes = gpu_pack(w, fw, h)
    assert np.array_equal(codes, wq)
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    bias_t = None if bias is None else dev(bias)
    if fp32_in:
        ws = torch.empty(max(1, B.fpq_gemm_workspace_size(M, N, K, 1)), dtype=torch.uint8, device=DEV)
        B.fpq_gemm(dev(x), 1, fx, sx, None, packed, fw, sw_t, bias_t, y, M, N, K, acc, ws)
    else:
        ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, K, 0)), dtype=torch.uint8, device=DEV)
        B.fpq_gemm(dev(xq), 0, fx, sx, None, packed, fw, sw_t, bias_t, y, M, N, K, acc, ws)
    torch.cuda.synchronize()
    return y.cpu().numpy(), (sx, xq, wq, sw)


LIN_SHAPES = [(256, 320, 320), (1, 16, 1), (5, 48, 3), (77, 768, 320), (130, 128, 65), (64, 2880, 96), (200, 1280, 130)]
PAIRS = [("E4M3", "E4M3"), ("E4M3", "E2M1"), ("E3M4", "E3M0"), ("E5M2", "E4M3"), ("E4M3", "E1M2"), ("E2M5", "E4M3_eq7"),
         ("E4M3_b9", "E2M1_b2"), ("E4M3", "E5M2")]


@pytest.mark.parametrize("M,K,N", LIN_SHAPES)
@pytest.mark.parametrize("fxn,fwn", PAIRS)
def test_linear_fp32_accumulate(M, K, N, fxn, fwn):
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    x = synth.activations((M, K), 1000 + M)
    w = synth.weights((N, K), 1500 + N)
    h = synth.rounding_mask((N, K), 1750 + N)
    bias = np.linspace(-1, 1, N).astype(np.float32)
    y, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP32, bias)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias)
    check_close(y, Y, T, what="linear %s x %s %s" % (fxn, fwn, (M, K, N)))


@pytest.mark.parametrize("M,K,N", LIN_SHAPES)
@pytest.mark.parametrize("fxn,fwn", [("E4M3", "E4M3"), ("E4M3", "E2M1"), ("E5M2", "E4M3"), ("E4M3", "E5M2"),
                                     ("E4M3_b9", "E2M1_b2")])
def test_linear_fp8_mfma(M, K, N, fxn, fwn):
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    x = synth.activations((M, K), 1000 + M)
    w = synth.weights((N, K), 1500 + N)
    h = synth.rounding_mask((N, K), 1750 + N)
    y, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP8_MFMA)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
    check_close(y, Y, T, rel=REL_FP8_MFMA, what="linear fp8-mfma %s x %s" % (fxn, fwn))


def test_linear_fp32_input_equals_codes_input():
    fx, fw = synth.E4M3, synth.E2M1
    for (M, K, N) in [(256, 320, 320), (9, 40, 17), (300, 72, 64)]:
        x = synth.activations((M, K), 5)
        w = synth.weights((N, K), 6)
        h = synth.rounding_mask((N, K), 7)
        y1, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP32, fp32_in=True)
        Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
        check_close(y1, Y, T, what="fp32-in %s" % ((M, K, N),))
        if K % 16 == 0:
            y0, _ = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP32)
            assert np.array_equal(y0, y1)


@pytest.mark.parametrize("acc", [B.FPQ_ACC_FP32, B.FPQ_ACC_FP8_MFMA])
@pytest.mark.parametrize("fwn", ["E4M3", "E2M1"])
def test_linear_exact_integers(acc, fwn):
    """Small-integer operands at scale 1: every product and partial sum is an exact integer below 2^24, so
    any summation order must reproduce the oracle with zero tolerance."""
    fx, fw = synth.E4M3, resolved(FORMATS[fwn])
    rng = np.random.default_rng(4)
    M, K, N = 130, 384, 72
    x = rng.choice(np.array([0, 1, 2, 3, 4, 5, 6, 7, 8, -1, -2, -3, -4, -6, -8], dtype=np.float32), (M, K))
    w = rng.choice(np.array([0, 1, 2, 3, 4, 6, -1, -2, -3, -4, -6], dtype=np.float32), (N, K))
    xq = oracle.quantize(x, fx, 1.0)
    sc = np.ones(N, dtype=np.float32)
    packed, sw_t, wq = gpu_pack(w, fw, None, sc)
    y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    B.fpq_gemm(dev(xq), 0, fx, 1.0, None, packed, fw, sw_t, None, y, M, N, K, acc)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy().astype(np.float64), x.astype(np.float64) @ w.astype(np.float64).T)
    # doubling sx doubles the output exactly
    y2 = torch.empty_like(y)
    B.fpq_gemm(dev(xq), 0, fx, 2.0, None, packed, fw, sw_t, None, y2, M, N, K, acc)
    torch.cuda.synchronize()
    assert torch.equal(y2, 2 * y)


@pytest.mark.parametrize("fxn,fwn", [("E4M3", "E4M3"), ("E4M3", "E2M1"), ("E3M4", "E3M0"), ("E5M2_eq7", "E1M2"),
                                     ("E4M3_eq7", "E2M5"), ("E4M3_bneg", "E3M2")])
def test_every_code_pair_decodes_exactly(fxn, fwn):
    """X holds activation code i alone in row i, W holds weight code j alone in row j: Y[i, j] is the product
    of the two decoded values, for all pairs of codes (single product: exact in fp32)."""
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    gx, gw = oracle.grid(fx), oracle.grid(fw)
    cx = [c | s for s in (0, 1 << (fx[0] + fx[1])) for c in range(len(gx)) if gx[c] <= fx[3]]
    cw = [c | s for s in (0, 1 << (fw[0] + fw[1])) for c in range(len(gw)) if gw[c] <= fw[3]]
    K = 16
    for pos in (0, 5, 15):
        xq = np.zeros((len(cx), K), dtype=np.uint8)
        xq[:, pos] = cx
        wvals = oracle.dequantize(np.array(cw, dtype=np.uint8), fw, 1.0).astype(np.float32)
        w = np.zeros((len(cw), K), dtype=np.float32)
        w[:, pos] = wvals
        sc = np.ones(len(cw), dtype=np.float32)
        packed, sw_t, wq = gpu_pack(w, fw, None, sc)
        assert np.array_equal(np.abs(oracle.dequantize(wq[:, pos], fw, 1.0)), np.abs(wvals.astype(np.float64)))
        y = torch.empty((len(cx), len(cw)), dtype=torch.float32, device=DEV)
        B.fpq_gemm(dev(xq), 0, fx, 1.0, None, packed, fw, sw_t, None, y, len(cx), len(cw), K, B.FPQ_ACC_FP32)
        torch.cuda.synchronize()
        want = np.outer(oracle.dequantize(np.array(cx, dtype=np.uint8), fx, 1.0), wvals.astype(np.float64))
        assert np.array_equal(y.cpu().numpy().astype(np.float64), want.astype(np.float32).astype(np.float64))


# ------------------------------------------------------------------------------ convolutions

def run_conv(x, w, h, fx, fw, stride, pad, acc, bias=None, fp32_in=False):
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, h)
    Bn, Cin, H, W = x.shape
    Cout, _, kh, kw = w.shape
    Ho, Wo = (H + 2 * pad - kh) // stride + 1, (W + 2 * pad - kw) // stride + 1
    packed, sw_t, codes = gpu_pack(w, fw, h)
    assert np.array_equal(codes, wq)
    y = torch.full((Bn, Cout, Ho, Wo), float("nan"), dtype=torch.float32, device=DEV)
    bias_t = None if bias is None else dev(bias)
    if fp32_in:
        ws = torch.empty(B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, kh, kw, stride, pad, 1), dtype=torch.uint8,
                         device=DEV)
        B.fpq_conv2d(dev(x), 1, fx, sx, None, packed, fw, sw_t, bias_t, y, Bn, Cin, H, W, Cout, kh, kw, stride, pad,
                     acc, ws)
    else:
        Cp = B.fpq_padded_channels(Cin)
        codes_nhwc = torch.empty(Bn * H * W * Cp, dtype=torch.uint8, device=DEV)
        B.fpq_quantize_nhwc(dev(x), fx, sx, None, codes_nhwc)
        ws = torch.empty(max(256, B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, kh, kw, stride, pad, 0)),
                         dtype=torch.uint8, device=DEV)
        B.fpq_conv2d(codes_nhwc, 0, fx, sx, None, packed, fw, sw_t, bias_t, y, Bn, Cin, H, W, Cout, kh, kw, stride,
                     pad, acc, ws)
    torch.cuda.synchronize()
    return y.cpu().numpy(), (sx, xq, wq, sw)


CONV_CASES = [  # B, Cin, H, W, Cout, k, stride, pad
    (1, 16, 8, 8, 32, 3, 1, 1), (2, 4, 9, 7, 5, 3, 1, 1), (1, 20, 6, 6, 33, 3, 2, 1), (2, 32, 5, 5, 64, 1, 1, 0),
    (1, 48, 12, 10, 130, 3, 1, 0), (3, 64, 7, 7, 4, 3, 1, 1), (1, 320, 16, 16, 96, 3, 1, 1), (2, 40, 8, 8, 40, 5, 1, 2),
    (1, 16, 9, 9, 16, 3, 3, 1),
]


@pytest.mark.parametrize("case", CONV_CASES)
@pytest.mark.parametrize("fxn,fwn,acc", [("E4M3", "E4M3", 0), ("E4M3", "E2M1", 0), ("E3M4", "E3M0", 0),
                                         ("E4M3", "E4M3", 1), ("E4M3", "E2M1", 1)])
def test_conv_small_full_compare(case, fxn, fwn, acc):
    Bn, Cin, H, W, Cout, k, stride, pad = case
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    x = synth.activations((Bn, Cin, H, W), 2000 + Cin)
    w = synth.weights((Cout, Cin, k, k), 2500 + Cout)
    h = synth.rounding_mask(w.shape, 2750 + Cout)
    bias = np.linspace(-0.5, 0.5, Cout).astype(np.float32)
    y, (sx, xq, wq, sw) = run_conv(x, w, h, fx, fw, stride, pad, acc, bias)
    Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, bias, stride=stride, pad=pad)
    check_close(y, Y, T, rel=REL_FP8_MFMA if acc else 1e-5, what="conv %s %s x %s acc %d" % (case, fxn, fwn, acc))


def test_conv_fp32_input_equals_codes_input():
    fx, fw = synth.E4M3, synth.E4M3
    x = synth.activations((2, 20, 9, 9), 1)
    w = synth.weights((24, 20, 3, 3), 2)
    h = synth.rounding_mask(w.shape, 3)
    y0, _ = run_conv(x, w, h, fx, fw, 1, 1, 0)
    y1, _ = run_conv(x, w, h, fx, fw, 1, 1, 0, fp32_in=True)
    assert np.array_equal(y0, y1)


@pytest.mark.parametrize("shape", [("linear", 256, 320, 320), ("linear", 9, 40, 17), ("linear", 2048, 1280, 320),
                                   ("linear", 8, 1280, 1280), ("linear", 16, 1024, 64), ("linear", 5, 48, 3), ("linear", 17, 1024, 64),
                                   ("conv", 2, 20, 9, 9, 24, 3, 1), ("conv", 1, 320, 32, 32, 320, 3, 1),
                                   ("conv", 2, 64, 16, 16, 160, 1, 2)])
def test_dynamic_scale_entry_equals_absmax_then_quantize(shape):
    """x_is_fp32 == 2: the scale absmax / maxval found inside the call gives the same codes, hence the same
    outputs bit for bit, as fpq_absmax followed by the fp32 entry with that device scale; and the result
    is the oracle's for the oracle's own absmax scale."""
    fx, fw = synth.E4M3, synth.E2M1
    if shape[0] == "linear":
        _, M, K, N = shape
        x = synth.activations((M, K), 11)
        w = synth.weights((N, K), 12)
    else:
        _, Bn, Cin, H, W, Cout, k, stride = shape
        x = synth.activations((Bn, Cin, H, W), 11)
        w = synth.weights((Cout, Cin, k, k), 12)
    x[0].flat[3] = -37.5    # the absmax element is negative
    h = synth.rounding_mask(w.shape, 13)
    packed, sw_t, wq = gpu_pack(w, fw, h)
    xd = dev(x)
    stat = torch.empty(2, dtype=torch.float32, device=DEV)
    tmp = torch.empty(1024, dtype=torch.float32, device=DEV)
    B.fpq_absmax(xd, fx[3], stat[0:1], stat[1:2], tmp)
    ys = []
    for mode in (1, 2):
        if shape[0] == "linear":
            y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
            ws = torch.empty(B.fpq_gemm_workspace_size(M, N, K, mode), dtype=torch.uint8, device=DEV)
            B.fpq_gemm(xd, mode, fx, 0.0, stat[1:2] if mode == 1 else None, packed, fw, sw_t, None, y, M, N, K,
                       B.FPQ_ACC_FP32, ws)
        else:
            pad = k // 2
            Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
            y = torch.full((Bn, Cout, Ho, Wo), float("nan"), dtype=torch.float32, device=DEV)
            ws = torch.empty(B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, k, k, stride, pad, mode), dtype=torch.uint8,
                             device=DEV)
            B.fpq_conv2d(xd, mode, fx, 0.0, stat[1:2] if mode == 1 else None, packed, fw, sw_t, None, y, Bn, Cin, H, W,
                         Cout, k, k, stride, pad, B.FPQ_ACC_FP32, ws)
        torch.cuda.synchronize()
        ys.append(y.cpu().numpy())
    assert np.array_equal(ys[0], ys[1])
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    assert sx == float(stat[1].item())
    xq = oracle.quantize(x, fx, sx)
    sw = sw_t.cpu().numpy()
    if shape[0] == "linear":
        Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
    else:
        Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, stride=stride, pad=k // 2)
    check_close(ys[1], Y, T, what="dynamic scale %s" % (shape,))


def test_conv_one_hot_taps_exact():
    """One non-zero input pixel and one non-zero weight tap: the output is a single 1 at the shifted position."""
    fx = fw = synth.E4M3
    Bn, Cin, H, W, Cout, k = 1, 16, 6, 5, 32, 3
    for ci, r, t, hi, wi in [(0, 0, 0, 0, 0), (15, 2, 1, 5, 4), (3, 1, 2, 2, 0), (7, 0, 2, 0, 4), (9, 1, 1, 3, 3)]:
        x = np.zeros((Bn, Cin, H, W), np.float32)
        w = np.zeros((Cout, Cin, k, k), np.float32)
        x[0, ci, hi, wi] = 1.0
        w[17, ci, r, t] = 1.0
        sc = np.ones(Cout, dtype=np.float32)
        packed, sw_t, _ = gpu_pack(w, fw, None, sc)
        codes = torch.empty(Bn * H * W * 16, dtype=torch.uint8, device=DEV)
        B.fpq_quantize_nhwc(dev(x), fx, 1.0, None, codes)
        y = torch.empty((Bn, Cout, H, W), dtype=torch.float32, device=DEV)
        B.fpq_conv2d(codes, 0, fx, 1.0, None, packed, fw, sw_t, None, y, Bn, Cin, H, W, Cout, k, k, 1, 1, 0)
        torch.cuda.synchronize()
        want = np.zeros((Bn, Cout, H, W), np.float32)
        ho, wo = hi + 1 - r, wi + 1 - t
        if 0 <= ho < H and 0 <= wo < W:
            want[0, 17, ho, wo] = 1.0
        assert np.array_equal(y.cpu().numpy(), want)


@pytest.mark.parametrize("kind,small", [("linear", False), ("linear", True), ("linear", None), ("conv", False)])
def test_dynamic_scale_of_an_all_zero_input(kind, small):
    """absmax = 0: the scale is 1 (not 0 / c), every code is +0 and the result is the bias."""
    fx, fw = synth.E4M3, synth.E2M1
    if kind == "linear":
        M, K, N = {False: (300, 320, 160), True: (8, 320, 160), None: (40, 320, 160)}[small]
        w = synth.weights((N, K), 91)
        x = torch.zeros((M, K), device=DEV)
    else:
        Bn, Cin, H, W, N = 2, 20, 9, 9, 33
        w = synth.weights((N, Cin, 3, 3), 92)
        x = torch.zeros((Bn, Cin, H, W), device=DEV)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    bias = np.linspace(-2, 2, N).astype(np.float32)
    if kind == "linear":
        y = torch.full((M, N), float("nan"), device=DEV)
        ws = torch.full((B.fpq_gemm_workspace_size(M, N, K, 2),), 0xEE, dtype=torch.uint8, device=DEV)
        B.fpq_gemm(x, B.FPQ_X_FP32_DYNAMIC, fx, 0.0, None, packed, fw, sw_t, dev(bias), y, M, N, K, B.FPQ_ACC_FP32, ws)
        want = np.broadcast_to(bias, (M, N))
        ncodes = M * K
    else:
        y = torch.full((Bn, N, H, W), float("nan"), device=DEV)
        ws = torch.full((B.fpq_conv2d_workspace_size(Bn, Cin, H, W, N, 3, 3, 1, 1, 2),), 0xEE, dtype=torch.uint8, device=DEV)
        B.fpq_conv2d(x, B.FPQ_X_FP32_DYNAMIC, fx, 0.0, None, packed, fw, sw_t, dev(bias), y, Bn, Cin, H, W, N, 3, 3, 1, 1,
                     B.FPQ_ACC_FP32, ws)
        want = np.broadcast_to(bias[None, :, None, None], (Bn, N, H, W))
        ncodes = Bn * H * W * B.fpq_padded_channels(Cin)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), want)
    h = ws.cpu().numpy()
    assert np.all(h[:ncodes] == 0)
    assert np.array_equal(h[-256:-248].view(np.float32), np.array([1.0, 0.0], dtype=np.float32))   # [scale, absmax]


@pytest.mark.parametrize("M,K,N", [(8, 1280, 1280), (8, 320, 1280), (16, 5120, 320), (1, 16, 1), (3, 48, 17), (13, 2576, 100),
                                     (16, 32, 16), (7, 8192, 33)])
@pytest.mark.parametrize("fwn", ["E4M3", "E2M1"])
def test_linear_with_at_most_sixteen_rows(M, K, N, fwn):
    """The kernel that splits K over the waves of a workgroup: ragged N, K not a multiple of 32, a K deep enough for
    several rounds of loads, bias, fp32 and codes input."""
    fx, fw = resolved(FORMATS["E4M3"]), resolved(FORMATS[fwn])
    x = synth.activations((M, K), 8000 + M + K)
    w = synth.weights((N, K), 8500 + N)
    h = synth.rounding_mask((N, K), 8750 + N) if fwn == "E2M1" else None
    bias = np.linspace(-1, 1, N).astype(np.float32)
    for fp32_in in (False, True):
        y, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP32, bias, fp32_in=fp32_in)
        Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias)
        check_close(y, Y, T, what="skinny linear %s" % ((M, K, N, fwn, fp32_in),))


@pytest.mark.parametrize("case", [("linear", 616, 768, 320), ("linear", 616, 768, 1280), ("linear", 512, 1280, 1280),
                                  ("linear", 33, 16, 31), ("linear", 100, 2560, 70), ("linear", 65, 1296, 97),
                                  ("conv", 8, 1280, 8, 8, 1280), ("conv", 3, 48, 5, 7, 33), ("conv", 2, 2560, 8, 8, 160)])
@pytest.mark.parametrize("fwn", ["E4M3", "E2M1"])
def test_small_outputs_with_short_k(case, fwn):
    """Small outputs with a short K, the shapes the plan sends to the register-staged kernels: the conditioning
    projections (M = 616), the layers of the 8 x 8 stage (M = 512), 1 x 1 convolutions, ragged M / N, odd K."""
    fx, fw = resolved(FORMATS["E4M3"]), resolved(FORMATS[fwn])
    if case[0] == "linear":
        _, M, K, N = case
        x = synth.activations((M, K), 8100 + M)
        w = synth.weights((N, K), 8600 + N)
        h = synth.rounding_mask((N, K), 8850 + N) if fwn == "E2M1" else None
        bias = np.linspace(-1, 1, N).astype(np.float32)
        y, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, B.FPQ_ACC_FP32, bias)
        Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias)
    else:
        _, Bn, Cin, H, W, Cout = case
        x = synth.activations((Bn, Cin, H, W), 8200 + Cin)
        w = synth.weights((Cout, Cin, 1, 1), 8700 + Cout)
        h = synth.rounding_mask(w.shape, 8950 + Cout) if fwn == "E2M1" else None
        bias = np.linspace(-0.5, 0.5, Cout).astype(np.float32)
        y, (sx, xq, wq, sw) = run_conv(x, w, h, fx, fw, 1, 0, B.FPQ_ACC_FP32, bias)
        Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, bias, stride=1, pad=0)
    check_close(y, Y, T, what="small output, short K %s" % ((case, fwn),))


def test_packed_header_check():
    w = synth.weights((40, 24, 3, 3), 5)
    packed, _, _ = gpu_pack(w, synth.E2M1, None, want_codes=False)
    assert B.fpq_packed_check(packed, 40, 24, 3, 3, synth.E2M1) == 0
    assert B.fpq_packed_check(packed, 40, 24, 3, 3, synth.E4M3) == -9          # another format
    assert B.fpq_packed_check(packed, 40, 24, 3, 3, (2, 1, 1, 4.0)) == -9      # another max value
    assert B.fpq_packed_check(packed, 41, 24, 3, 3, synth.E2M1) == -9
    assert B.fpq_packed_check(packed, 40, 24, 1, 1, synth.E2M1) == -9
    assert B.fpq_packed_check(torch.zeros(512, dtype=torch.uint8, device=DEV), 40, 24, 3, 3, synth.E2M1) == -9
    assert B.fpq_packed_check(packed, 40, 24, 3, 3, (2, 1, 1, 5.0)) == -2      # not a format at all


def test_fp32_input_with_more_rows_than_a_grid_dimension_and_padded_k():
    """M > 65535 rows and K not a multiple of 16: the channels-last quantizer walks the rows in several rounds."""
    M, K, N = 70001, 24, 8
    fx = fw = synth.E4M3
    x = synth.activations((M, K), 77)
    w = synth.weights((N, K), 78)
    sx, xq, wq, sw = oracle_linear_inputs(x, w, None, fx, fw)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    y = torch.full((M, N), float("nan"), device=DEV)
    ws = torch.empty(B.fpq_gemm_workspace_size(M, N, K, 1), dtype=torch.uint8, device=DEV)
    B.fpq_gemm(dev(x), 1, fx, sx, None, packed, fw, sw_t, None, y, M, N, K, B.FPQ_ACC_FP32, ws)
    torch.cuda.synchronize()
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
    check_close(y.cpu().numpy(), Y, T, what="70001-row fp32 input")
    codes = ws.cpu().numpy()[:M * 32].reshape(M, 32)
    assert np.array_equal(codes[:, :K], xq) and np.all(codes[:, K:] == 0)


@pytest.mark.parametrize("N", [2080, 1928])
def test_output_with_more_than_two_to_the_31_elements(N):
    """M * N > 2^32 (a 17 GB fp32 result; N = 2080 runs the large-tile kernel, 1928 the small-tile one): element
    offsets must be 64-bit everywhere.  Compared with the oracle on whole rows: the first and the last ones, the
    rows either side of elements 2^30, 2^31 and 2^32, and random ones."""
    M, K = 2230001, 16
    fx = fw = synth.E4M3
    x = synth.activations((M, K), 91)
    w = synth.weights((N, K), 92)
    bias = np.linspace(-1, 1, N).astype(np.float32)
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    wq, sw = oracle.pack_weights(w, fw, None)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    y.fill_(float("nan"))
    ws = torch.empty(B.fpq_gemm_workspace_size(M, N, K, 1), dtype=torch.uint8, device=DEV)
    assert 2 ** 32 // N + 1 < M
    print("launch M=%d N=%d K=%d" % (M, N, K), flush=True)
    B.fpq_gemm(dev(x), 1, fx, sx, None, packed, fw, sw_t, dev(bias), y, M, N, K, B.FPQ_ACC_FP32, ws)
    torch.cuda.synchronize()
    assert not bool(torch.isnan(y).any())
    r30, r31, r32 = 2 ** 30 // N, 2 ** 31 // N, 2 ** 32 // N
    rows = sorted(set([0, 1, 127, 128, M - 130, M - 2, M - 1, r30 - 1, r30, r30 + 1, r31 - 1, r31, r31 + 1, r32 - 1, r32,
                       r32 + 1] +
                      list(np.random.default_rng(93).integers(0, M, 40))))
    got = y[torch.tensor(rows, device=DEV)].cpu().numpy()
    del y
    Y, T = oracle.gemm(oracle.quantize(x[rows], fx, sx), fx, sx, wq, fw, sw, bias)
    check_close(got, Y, T, what="rows of a %d x %d result" % (M, N))


@pytest.mark.parametrize("Cout", [320, 328])
def test_conv_output_with_more_than_two_to_the_32_elements(Cout):
    """The same for the NCHW result of a convolution (B * Cout * Ho * Wo > 2^32; 320 channels run the large-tile
    kernel, 328 the small-tile one): whole images compared, among them those that hold elements 2^31 and 2^32."""
    Bn, Cin, H, W, k = 830, 4, 128, 128, 3
    fx = fw = synth.E4M3
    x = synth.activations((Bn, Cin, H, W), 94)
    w = synth.weights((Cout, Cin, k, k), 95)
    bias = np.linspace(-1, 1, Cout).astype(np.float32)
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    wq, sw = oracle.pack_weights(w, fw, None)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    per_image = Cout * H * W
    assert Bn * per_image > 2 ** 32
    y = torch.empty((Bn, Cout, H, W), dtype=torch.float32, device=DEV)
    y.fill_(float("nan"))
    ws = torch.empty(B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, k, k, 1, 1, 1), dtype=torch.uint8, device=DEV)
    print("launch B=%d Cout=%d" % (Bn, Cout), flush=True)
    B.fpq_conv2d(dev(x), 1, fx, sx, None, packed, fw, sw_t, dev(bias), y, Bn, Cin, H, W, Cout, k, k, 1, 1,
                 B.FPQ_ACC_FP32, ws)
    torch.cuda.synchronize()
    assert not bool(torch.isnan(y).any())
    images = sorted({0, 2 ** 30 // per_image, 2 ** 31 // per_image, 2 ** 32 // per_image, Bn - 1})
    got = y[torch.tensor(images, device=DEV)].cpu().numpy()
    del y
    Y, T = oracle.conv2d(oracle.quantize(x[images], fx, sx), fx, sx, wq, fw, sw, bias, stride=1, pad=1)
    check_close(got, Y, T, what="images %s of a %d-image result" % (images, Bn))


# ------------------------------------------------------------------------------ large-tile (N % 160 == 0) kernels

@pytest.mark.parametrize("M,K,N", [(256, 128, 160), (257, 144, 160), (300, 2880, 320), (1000, 320, 480), (512, 6400, 160),
                                     (4096, 64, 320)])
@pytest.mark.parametrize("fxn,fwn,acc", [("E4M3", "E4M3", 0), ("E4M3", "E2M1", 0), ("E3M4", "E3M0", 0), ("E3M4", "E2M5", 0),
                                         ("E4M3", "E4M3", 1), ("E4M3", "E2M1", 1)])
def test_linear_large_tile_and_split_k(M, K, N, fxn, fwn, acc):
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    x = synth.activations((M, K), 3000 + M)
    w = synth.weights((N, K), 3500 + N)
    h = synth.rounding_mask((N, K), 3750 + N)
    bias = np.linspace(-1, 1, N).astype(np.float32)
    y, (sx, xq, wq, sw) = run_linear(x, w, h, fx, fw, acc, bias)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias)
    check_close(y, Y, T, rel=REL_FP8_MFMA if acc else 1e-5, what="large-tile linear %s" % ((M, K, N, fxn, fwn, acc),))


@pytest.mark.parametrize("case", [(1, 32, 16, 16, 160, 3, 1, 1), (2, 48, 13, 11, 320, 3, 1, 1), (4, 160, 9, 9, 160, 3, 2, 1),
                                  (1, 640, 16, 16, 160, 3, 1, 1), (3, 20, 10, 10, 160, 1, 1, 0), (1, 16, 40, 40, 160, 5, 1, 2)])
@pytest.mark.parametrize("fxn,fwn,acc", [("E4M3", "E4M3", 0), ("E4M3", "E2M1", 0), ("E3M4", "E3M0", 0), ("E4M3", "E2M1", 1)])
def test_conv_large_tile_and_split_k(case, fxn, fwn, acc):
    Bn, Cin, H, W, Cout, k, stride, pad = case
    fx, fw = resolved(FORMATS[fxn]), resolved(FORMATS[fwn])
    x = synth.activations((Bn, Cin, H, W), 4000 + Cin)
    w = synth.weights((Cout, Cin, k, k), 4500 + Cout)
    h = synth.rounding_mask(w.shape, 4750 + Cout)
    bias = np.linspace(-0.5, 0.5, Cout).astype(np.float32)
    y, (sx, xq, wq, sw) = run_conv(x, w, h, fx, fw, stride, pad, acc, bias)
    Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, bias, stride=stride, pad=pad)
    check_close(y, Y, T, rel=REL_FP8_MFMA if acc else 1e-5, what="large-tile conv %s" % ((case, fxn, fwn, acc),))


# ------------------------------------------------------------------------------ separately quantized concatenation

@pytest.mark.parametrize("case", [("conv", 2, 24, 40, 9, 9, 48, 3), ("conv", 1, 320, 640, 32, 32, 320, 1),
                                  ("conv", 2, 640, 640, 8, 8, 320, 3), ("linear", 300, 64, 96, 130),
                                  ("linear", 512, 2560, 2560, 320)])
@pytest.mark.parametrize("acc", [B.FPQ_ACC_FP32, B.FPQ_ACC_FP8_MFMA])
def test_concatenated_input_with_one_scale_per_part(case, acc):
    """Section VI-A: the two halves of a channel-wise concatenation are quantized separately, each with its own
    per-tensor scale.  One call per half on that half's codes and weight slice, the second adding to y
    (FPQ_OUT_ACCUMULATE), must give the sum of the oracle's two layers."""
    fx, fw = synth.E4M3, synth.E4M3
    if case[0] == "conv":
        _, Bn, Ca, Cb, H, W, Cout, k = case
        a = synth.activations((Bn, Ca, H, W), 21)
        b = (synth.activations((Bn, Cb, H, W), 22) * np.float32(7.0)).astype(np.float32)   # another value range
        w = synth.weights((Cout, Ca + Cb, k, k), 23)
        parts = [(a, w[:, :Ca].copy()), (b, w[:, Ca:].copy())]
        N = Cout
    else:
        _, M, Ka, Kb, N = case
        a = synth.activations((M, Ka), 21)
        b = (synth.activations((M, Kb), 22) * np.float32(7.0)).astype(np.float32)
        w = synth.weights((N, Ka + Kb), 23)
        parts = [(a, w[:, :Ka].copy()), (b, w[:, Ka:].copy())]
    # one weight scale per output channel over the whole (concatenated) row
    sw = (np.abs(w.reshape(N, -1)).max(axis=1) / np.float32(fw[3])).astype(np.float32)
    bias = np.linspace(-0.5, 0.5, N).astype(np.float32)
    y = None
    Ysum, Tsum = 0.0, 0.0
    for idx, (x, wp) in enumerate(parts):
        sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
        xq = oracle.quantize(x, fx, sx)
        wq, sw_o = oracle.pack_weights(wp, fw, None, sw)
        packed, sw_t, _ = gpu_pack(wp, fw, None, sw)
        flags = acc | (B.FPQ_OUT_ACCUMULATE if idx else 0)
        bias_t = dev(bias) if idx == 0 else None
        if case[0] == "conv":
            Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw_o, bias if idx == 0 else None, stride=1, pad=k // 2)
            if y is None:
                y = torch.full((Bn, Cout, H, W), float("nan"), dtype=torch.float32, device=DEV)
            ws = torch.empty(B.fpq_conv2d_workspace_size(Bn, x.shape[1], H, W, Cout, k, k, 1, k // 2, 1), dtype=torch.uint8,
                             device=DEV)
            B.fpq_conv2d(dev(x), 1, fx, sx, None, packed, fw, sw_t, bias_t, y, Bn, x.shape[1], H, W, Cout, k, k, 1, k // 2,
                         flags, ws)
        else:
            Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw_o, bias if idx == 0 else None)
            if y is None:
                y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
            ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, x.shape[1], 1)), dtype=torch.uint8, device=DEV)
            B.fpq_gemm(dev(x), 1, fx, sx, None, packed, fw, sw_t, bias_t, y, M, N, x.shape[1], flags, ws)
        Ysum = Ysum + Y
        Tsum = Tsum + T
    torch.cuda.synchronize()
    check_close(y.cpu().numpy(), Ysum, Tsum, rel=REL_FP8_MFMA if acc else 1e-5, what="split concat %s acc %d" % (case, acc))


# ------------------------------------------------------------------------------ what the FP8-MFMA mode computes

def _two_term_gemm(xrow, wrow, acc):
    """One output: sum_k xrow[k] * wrow[k], all values on the E4M3 grid, scales 1, K = 16."""
    f = synth.E4M3
    M = N = 16
    x = np.zeros((M, 16), dtype=np.float32)
    w = np.zeros((N, 16), dtype=np.float32)
    x[3], w[5] = xrow, wrow
    xq = oracle.quantize(x, f, 1.0)
    assert np.array_equal(oracle.dequantize(xq, f, 1.0), x)          # on the grid: the codes hold the values exactly
    packed, sw_t, wq = gpu_pack(w, f, None, np.ones(N, dtype=np.float32))
    assert np.array_equal(oracle.dequantize(wq, f, 1.0), w)
    y = torch.empty((M, N), dtype=torch.float32, device=DEV)
    B.fpq_gemm(dev(xq), 0, f, 1.0, None, packed, f, sw_t, None, y, M, N, 16, acc)
    torch.cuda.synchronize()
    yh = y.cpu().numpy()
    assert np.count_nonzero(yh) <= 1
    return float(yh[3, 5])


def test_fp8_mfma_mode_drops_low_product_bits_and_fp32_mode_does_not():
    """The reason for the two accumulate modes, shown through the ABI.  The 8-bit matrix instruction aligns the
    products of each group of 8 consecutive k to the group's largest exponent and drops bits more than 13 binary
    places below it; only the group sums are added in fp32.  FPQ_ACC_FP32 (codes expanded to bf16, bf16 matrix
    instruction) returns the exact sums."""
    z = [0.0] * 14
    # 64 * 64 + 0.5 * 0.5 in one group of 8: 0.25 lies 14 places below 4096
    assert _two_term_gemm([64, 0.5] + z, [64, 0.5] + z, B.FPQ_ACC_FP32) == 4096.25
    assert _two_term_gemm([64, 0.5] + z, [64, 0.5] + z, B.FPQ_ACC_FP8_MFMA) == 4096.0
    # 0.5 (13 places below) survives
    assert _two_term_gemm([64, 1] + z, [64, 0.5] + z, B.FPQ_ACC_FP8_MFMA) == 4096.5
    # 4096 - 4096 + 1.75: the last bit of 1.75 is cut although the large terms cancel
    assert _two_term_gemm([64, 64, 1.75] + z[:13], [64, -64, 1] + z[:13], B.FPQ_ACC_FP32) == 1.75
    assert _two_term_gemm([64, 64, 1.75] + z[:13], [64, -64, 1] + z[:13], B.FPQ_ACC_FP8_MFMA) == 1.5
    # the same two terms in different groups of 8 (k = 0 and k = 8) are added in fp32: exact in both modes
    far = [64] + [0.0] * 7 + [0.5] + [0.0] * 7
    assert _two_term_gemm(far, far, B.FPQ_ACC_FP8_MFMA) == 4096.25
    assert _two_term_gemm(far, far, B.FPQ_ACC_FP32) == 4096.25


def test_fp8_mfma_mode_misses_the_layer_tolerance_on_the_synthetic_workload():
    """Configuration 1 (256 x 320 x 320, activations with x20 outliers) in both modes against the tolerance the layer
    results must meet, 1e-5 * sum|a_k b_k| + 1e-6: the fp32-accumulate mode meets it everywhere, the FP8-MFMA mode
    misses it on a visible share of the outputs (which is why that mode is an option outside the tolerance and the
    benchmark's headline runs in the other one)."""
    fx, fw = synth.E4M3, synth.E4M3
    x = synth.activations((256, 320), 1000)
    w = synth.weights((320, 320), 1500)
    y32, (sx, xq, wq, sw) = run_linear(x, w, None, fx, fw, B.FPQ_ACC_FP32)
    y8, _ = run_linear(x, w, None, fx, fw, B.FPQ_ACC_FP8_MFMA)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
    tol = 1e-5 * T + 1e-6
    assert not (np.abs(y32 - Y) > tol).any()
    miss = float((np.abs(y8 - Y) > tol).mean())
    worst = float((np.abs(y8 - Y) / tol).max())
    print("FP8-MFMA mode: %.2f %% of outputs outside 1e-5 T + 1e-6, worst err/tol %.1f" % (100 * miss, worst))
    assert 0.001 < miss < 0.2 and worst < 85.0      # 7 * 2^-13 / 1e-5 = 85 is the mode's own bound


@pytest.mark.parametrize("of", [list, lambda f: B.fmt(f), lambda f: np.array(f, dtype=np.float32),
                                lambda f: np.array(f, dtype=np.float64), lambda f: torch.tensor(f),
                                lambda f: (np.int64(f[0]), np.int32(f[1]), f[2], np.float32(f[3]))])
def test_a_format_is_anything_with_its_four_elements(of):
    """Also an array whose buffer happens to have the size of the C structure."""
    x = dev(synth.activations((1000,), 4321))
    want, got = (torch.zeros(1000, dtype=torch.uint8, device=DEV) for _ in range(2))
    B.fpq_quantize(x, synth.E4M3, 0.5, None, want)
    B.fpq_quantize(x, of(synth.E4M3), 0.5, None, got)
    torch.cuda.synchronize()
    assert torch.equal(got, want)


@pytest.mark.parametrize("fx,fw", [((3, 4, 3, 0.0), (2, 5, -48, 0.0)), ((3, 4, -40, 0.0), (3, 0, 4, 0.0)), ((2, 5, 48, 0.0), (2, 5, 48, 0.0)),
                                   ((3, 4, 16, 0.0), (2, 5, -16, 0.0))])
def test_formats_of_far_out_biases_on_far_out_scales(fx, fw):
    """Large activations on small weights: the scales make up for each other, and for what the formats' biases add to them."""
    fx, fw = resolved(fx), resolved(fw)
    M, K, N = 70, 256, 48
    x = synth.activations((M, K), 5000) * np.float32(2.0 ** 60)
    w = synth.weights((N, K), 5001) * np.float32(2.0 ** -60)
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, None)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw)
    packed, sw_t, _ = gpu_pack(w, fw, None)
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, K, 0)), dtype=torch.uint8, device=DEV)
    B.fpq_gemm(dev(xq), 0, fx, sx, None, packed, fw, sw_t, None, y, M, N, K, 0, ws)
    torch.cuda.synchronize()
    check_close(y.cpu().numpy(), Y, T, what="%s %s" % (fx, fw))
