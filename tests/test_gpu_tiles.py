"""The tiles for small problems and for widths that are no multiple of 160 (64 x 64 with K split over the wavefronts,
128 x 64, 128 x 128, and 128 x 160 with a ragged last column), at their edges, against the oracle: remainders of rows,
columns and K, images that end inside a lane's four pixels, accumulating and sliced forms, and results as codes.
Of shapes with one row of at most 320 codes per output, the accumulating call alone takes a tile: stored, and as codes, they are
mostly the short-K kernel's (test_gpu_strip.py); test_unsliced_tiles_just_beyond_the_short_k has the tiles there."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, check_close, dev, gpu_pack
from test_gpu_codes_out import test_linear_activation_then_codes as linear_activation_case
from test_gpu_codes_out import test_conv_silu_then_codes as conv_silu_case

pytestmark = pytest.mark.gpu

E4M3, E2M1, E3M4, E3M0 = synth.E4M3, synth.E2M1, synth.E3M4, synth.E3M0
FORMS = [(E4M3, E4M3, 0), (E4M3, E2M1, 0), (E4M3, E4M3, 1), (E4M3, E2M1, 1), (E3M4, E3M4, 0), (E3M4, E3M0, 0)]
REL_FP8_MFMA = 7 * 2.0 ** -13

LINEAR = [(17, 1024, 1), (64, 1040, 64), (65, 1152, 66), (200, 2048, 333),           # K over the wavefronts, four stages
          (40, 5120, 130), (273, 2768, 72), (17, 16384, 33),                         # ... and over slices
          (1407, 3312, 749), (2049, 1024, 516),                                      # ... two stages
          (4097, 336, 700), (9000, 16, 300), (8961, 144, 300), (9000, 400, 301),     # 128 x 64
          (4918, 1040, 896), (4864, 272, 895),                                       # 128 x 128
          (8193, 144, 1116),                                                         # 128 x 160, ragged last column
          # larger grids, by results and operands: 128 x 64 / 128 x 128 / 128 x 160 for fp32 results of hardware encodings ...
          (9772, 1040, 516), (19112, 1024, 301), (9772, 272, 1116), (12222, 272, 895), (7812, 272, 1100), (12222, 336, 749),
          # ... and of halves
          (12222, 1024, 301), (9772, 144, 749), (9772, 144, 895)]


@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("M,K,N", LINEAR)
def test_linear(M, K, N, fx, fw, acc):
    print(M, K, N, fx, fw, acc, flush=True)
    x = synth.activations((M, K), 400 + M)
    w = synth.weights((N, K), 500 + N)
    bias = np.linspace(-1, 1, N).astype(np.float32) if N % 2 else None
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, None)
    rows = np.unique(np.concatenate([np.arange(min(M, 70)), np.arange(max(0, M - 70), M),
                                     np.random.default_rng(M).integers(0, M, 120)]))
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias, rows=rows)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, K, 0)), dtype=torch.uint8, device=DEV)
    buf = torch.full((M * N + 8,), float("nan"), dtype=torch.float32, device=DEV)
    y = buf[4:4 + M * N].view(M, N)
    run = lambda flag: B.fpq_gemm(dev(xq), 0, fx, sx, None, packed, fw, sw_t, None if bias is None else dev(bias), y, M, N, K,
                                  acc | flag, ws)
    run(0)
    torch.cuda.synchronize()
    once = y.cpu().numpy().copy()
    assert not np.isnan(once).any(), "unwritten outputs"
    rel = REL_FP8_MFMA if acc else 1e-5
    check_close(once[rows], Y, T, rel=rel, what="linear")
    y.fill_(1.0)
    run(B.FPQ_OUT_ACCUMULATE)
    torch.cuda.synchronize()
    h = buf.cpu().numpy()
    assert np.isnan(h[:4]).all() and np.isnan(h[-4:]).all(), "written outside the result"
    assert np.allclose(h[4:-4].reshape(M, N), once + np.float32(1), rtol=1e-6, atol=1e-6 * np.abs(once).max())


CONV = [(2, 128, 19, 19, 36, 3, 1, 1), (1, 128, 3, 3, 70, 3, 1, 1), (5, 1040, 1, 1, 70, 1, 1, 0), (9, 128, 3, 1, 20, 3, 1, 1),
        (2, 200, 35, 33, 72, 3, 2, 1), (1, 64, 13, 7, 50, 5, 1, 2), (1, 1440, 15, 7, 66, 3, 1, 1), (3, 130, 9, 9, 65, 3, 1, 0),
        (2, 128, 70, 71, 130, 3, 1, 1), (1, 320, 32, 64, 320, 3, 1, 1),
        (3, 36, 67, 65, 200, 3, 1, 1), (3, 20, 133, 130, 196, 3, 2, 1), (2800, 16, 2, 2, 197, 1, 1, 0),
        (3, 20, 81, 81, 250, 3, 1, 1), (3, 16, 67, 65, 1116, 1, 1, 0), (2, 320, 32, 32, 320, 3, 1, 1),
        (3, 128, 64, 64, 301, 3, 1, 1), (2, 16, 70, 70, 749, 3, 1, 1), (2, 16, 63, 62, 516, 1, 1, 0)]      # 128 x 64, 128, 160


@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("case", CONV)
def test_conv(case, fx, fw, acc):
    print(case, fx, fw, acc, flush=True)
    Bn, Cin, H, W, Cout, k, stride, pad = case
    x = synth.activations((Bn, Cin, H, W), 600 + Cin)
    w = synth.weights((Cout, Cin, k, k), 700 + Cout)
    bias = np.linspace(-0.5, 0.5, Cout).astype(np.float32) if Cout % 4 else None
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, None)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    codes = torch.empty(Bn * H * W * B.fpq_padded_channels(Cin), dtype=torch.uint8, device=DEV)
    B.fpq_quantize_nhwc(dev(x), fx, sx, None, codes)
    Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, bias, stride=stride, pad=pad)
    ws = torch.empty(max(256, B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, k, k, stride, pad, 0)), dtype=torch.uint8,
                     device=DEV)
    buf = torch.full((Y.size + 8,), float("nan"), dtype=torch.float32, device=DEV)
    y = buf[4:4 + Y.size]
    run = lambda flag: B.fpq_conv2d(codes, 0, fx, sx, None, packed, fw, sw_t, None if bias is None else dev(bias), y, Bn, Cin,
                                    H, W, Cout, k, k, stride, pad, acc | flag, ws)
    run(0)
    torch.cuda.synchronize()
    once = y.cpu().numpy().reshape(Y.shape).copy()
    assert not np.isnan(once).any(), "unwritten outputs"
    check_close(once, Y, T, rel=REL_FP8_MFMA if acc else 1e-5, what="conv")
    y.fill_(1.0)
    run(B.FPQ_OUT_ACCUMULATE)
    torch.cuda.synchronize()
    h = buf.cpu().numpy()
    assert np.isnan(h[:4]).all() and np.isnan(h[-4:]).all(), "written outside the result"
    assert np.allclose(h[4:-4].reshape(Y.shape), once + np.float32(1), rtol=1e-6, atol=1e-6 * np.abs(once).max())


@pytest.mark.parametrize("fw,fy,acc", [(E4M3, E4M3, 0), (E2M1, E3M4, 0), (E4M3, E4M3, 1)])
@pytest.mark.parametrize("act", ["silu", "geglu"])
@pytest.mark.parametrize("M,K,N", [(65, 1152, 96), (40, 5120, 128), (1407, 3312, 736), (4097, 336, 704), (4918, 1024, 896),
                                   (8193, 144, 1088), (4990, 400, 2048), (12222, 400, 896), (4990, 1024, 2048)])
def test_linear_codes_out(M, K, N, fw, fy, acc, act):
    linear_activation_case(M, K, N, fw, fy, acc, act)


@pytest.mark.parametrize("case", [(2, 128, 19, 19, 36, 3, 1, 1), (1, 1440, 15, 7, 66, 3, 1, 1), (2, 128, 70, 71, 130, 3, 1, 1),
                                  (3, 36, 67, 65, 200, 3, 1, 1), (3, 20, 81, 81, 250, 3, 1, 1), (2, 16, 63, 62, 749, 1, 1, 0),
                                  (2, 16, 70, 70, 1100, 3, 1, 1), (2, 16, 63, 62, 1116, 3, 1, 1)])
def test_conv_codes_out(case):
    conv_silu_case(case)


@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("M,K,N", [(8193, 400, 1116), (9772, 400, 749), (9772, 400, 895), (8200, 336, 640)])
def test_unsliced_tiles_just_beyond_the_short_k(M, K, N, fx, fw, acc):
    """128 x 160 with a ragged last column, 128 x 128 and 128 x 160 of halves, 128 x 160 with ragged rows."""
    test_linear(M, K, N, fx, fw, acc)


@pytest.mark.parametrize("fw,fy,acc", [(E4M3, E4M3, 0), (E2M1, E3M4, 0), (E4M3, E4M3, 1)])
@pytest.mark.parametrize("act", ["silu", "geglu"])
@pytest.mark.parametrize("M,K,N", [(8192, 400, 320), (8200, 336, 640)])
def test_codes_of_128_x_160_tiles_just_beyond_the_short_k(M, K, N, fw, fy, acc, act):
    linear_activation_case(M, K, N, fw, fy, acc, act)


def test_conv_codes_of_128_x_160_tiles_just_beyond_the_short_k():
    conv_silu_case((8, 336, 32, 32, 320, 1, 1, 0))


@pytest.mark.parametrize("fx,fw,acc", FORMS)
def test_grouped_call_has_the_bits_of_single_calls(fx, fw, acc):
    """Problems of the 64 x 64 tile next to problems whose K is split over the wavefronts."""
    shapes = [(616, 768, 1280)] * 4 + [(616, 768, 640), (616, 320, 100), (200, 1280, 130), (200, 1040, 1), (17, 2048, 65)]
    ps = []
    for i, (M, K, N) in enumerate(shapes):
        x = synth.activations((M, K), 800 + i)
        sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
        packed, sw_t, _ = gpu_pack(synth.weights((N, K), 900 + i), fw, None, want_codes=False)
        ps.append((dev(oracle.quantize(x, fx, sx)), dev(np.array([sx], dtype=np.float32)), packed, sw_t,
                   dev(np.linspace(-1, 1, N).astype(np.float32)), torch.full((M, N), float("nan"), device=DEV), M, N, K))
    B.fpq_gemm_grouped(B.gemm_problems(ps), B.FPQ_X_CODES, fx, fw, acc, None)
    torch.cuda.synchronize()
    for xq, sx, packed, sw_t, bias, y, M, N, K in ps:
        ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, K, 0)), dtype=torch.uint8, device=DEV)
        y1 = torch.full_like(y, float("nan"))
        B.fpq_gemm(xq, 0, fx, 0.0, sx, packed, fw, sw_t, bias, y1, M, N, K, acc, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, y1), (M, K, N)


# Operands that are decoded arithmetically on widths that are multiples of 160: the 128 x 160 tile in 11, 5, 2 and one slices, the
# 256 x 160 tile, and the register-staged kernel for a small output or a small grid with a short K.
@pytest.mark.parametrize("fx,fw", [(synth.E5M2, synth.E5M2), (E4M3, synth.E5M2), (synth.E5M2, E2M1)])
@pytest.mark.parametrize("M,K,N", [(256, 11520, 1280), (40, 5120, 1280), (4096, 2880, 320), (2048, 1280, 1280), (4096, 640, 640),
                                   (3072, 2048, 2560), (616, 768, 320)])
def test_arithmetic_operands(M, K, N, fx, fw):
    test_linear(M, K, N, fx, fw, 0)


@pytest.mark.parametrize("M,K,N", [(200, 1040, 192), (200, 1040, 193), (200, 1024, 192), (616, 1024, 320), (1407, 3312, 100)])
def test_grouped_bits_do_not_depend_on_the_other_problems(M, K, N):
    """At and beyond the 12 tiles, above and at the 8 steps of K up to which a problem does not have its K split over the wavefronts;
    alone, and among problems that fill the chip."""
    def problem(M, K, N, seed):
        x = synth.activations((M, K), seed)
        sx = oracle.scale_from_absmax(oracle.absmax(x), E4M3[3])
        packed, sw_t, _ = gpu_pack(synth.weights((N, K), seed + 1), E4M3, None, want_codes=False)
        return [dev(oracle.quantize(x, E4M3, sx)), dev(np.array([sx], dtype=np.float32)), packed, sw_t, None,
                torch.full((M, N), float("nan"), device=DEV), M, N, K]
    one, other = problem(M, K, N, 950), problem(616, 1024, 320, 960)
    B.fpq_gemm_grouped(B.gemm_problems([one]), B.FPQ_X_CODES, E4M3, E4M3, 0, None)
    torch.cuda.synchronize()
    alone = one[5].clone()
    one[5].fill_(float("nan"))
    others = [other[:5] + [torch.empty_like(other[5])] + other[6:] for _ in range(20)]
    B.fpq_gemm_grouped(B.gemm_problems(others[:7] + [one] + others[7:]), B.FPQ_X_CODES, E4M3, E4M3, 0, None)
    torch.cuda.synchronize()
    assert torch.equal(one[5], alone)
