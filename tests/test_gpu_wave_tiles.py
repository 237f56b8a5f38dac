"""The 128 x 80 and 64 x 80 tiles with K split over the wavefronts, at their edges, against the oracle: remainders of rows, columns and
K, fewer steps of 64 codes than wavefronts, rows and columns that are a fraction of a tile, channels that wrap several taps a step, images that
end inside a lane's four pixels, results that are added.  The rule, compiled here for the host, and the library's query are asked which of the
two tiles each shape takes in the encodings of the hardware, and which where both operands are moved into halves."""
import functools
import os
import subprocess
import tempfile

import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, check_close, dev, gpu_pack

E4M3, E2M1, E3M4, E3M0 = synth.E4M3, synth.E2M1, synth.E3M4, synth.E3M0
FORMS = [(E4M3, E4M3), (E4M3, E2M1), (E3M4, E3M4), (E3M4, E3M0)]
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2408_06995_amd", "csrc")
PROGRAM = r"""
#include <stdio.h>
#include "fpq_host.h"
using namespace fpq;
int main()
{
    // the divisions of the kernels: around every multiple, at the ends of the range
    const long long top = (1ll << 31) - 1;
    for (long long d : {1ll, 2ll, 3ll, 5ll, 7ll, 16ll, 53ll, 64ll, 80ll, 961ll, 4096ll, 65535ll, 65536ll, 1000003ll, (1ll << 30) - 1, 1ll << 30, top - 1, top}) {
        const Divisor by = divisor(d);
        for (long long q = 0; q * d <= top; q += q < 1000 ? 1 : q / 7 + 1)
            for (long long n = q * d - 1; n <= q * d + 1; ++n)
                if (n >= 0 && n <= top && (long long)((((unsigned long long)(2 * n) * by.mul) >> 32) >> by.shift) != n / d)
                    return printf("%lld / %lld\n", n, d), 1;
    }
    long long M, N, K;
    int form, ragged;
    while (scanf("%lld %lld %lld %d %d", &M, &N, &K, &form, &ragged) == 5) {
        const GemmPlan p = plan_gemm(M, N, (K + 127) / 128 * 128, (PlanForm)form);
        printf("%d\n", plan_over_waves(p, M, N, K, (PlanForm)form, ragged != 0).tile);
    }
    return 0;
}
"""
LINEAR, CONV, HALF = 0, 1, 4          # PlanForm
T128, T64 = 7, 8                      # GemmTile


@functools.lru_cache(maxsize=None)
def program():
    d = tempfile.mkdtemp()
    with open(os.path.join(d, "rule.cpp"), "w") as f:
        f.write(PROGRAM)
    exe = os.path.join(d, "rule")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, os.path.join(d, "rule.cpp"),
                           "-o", exe])
    return exe


def tile_of(M, N, K, form, ragged=False):
    return int(subprocess.run([program()], input="%d %d %d %d %d\n" % (M, N, K, form, ragged), capture_output=True, text=True,
                              check=True).stdout)


def test_divisions_and_what_keeps_its_plan():
    assert tile_of(4096, 320, 2880, CONV) == T64 and tile_of(2048, 1280, 11520, CONV) == T128 and tile_of(2048, 1280, 11520, HALF) == T128
    for M, N, K, form in [(32768, 320, 5760, CONV), (32768, 320, 1280, LINEAR), (64, 320, 11520, CONV), (8, 1280, 1280, LINEAR),
                          (2048, 1280, 11520, 2), (2048, 1280, 11520, 3)]:                 # the last two: results as codes
        assert tile_of(M, N, K, form) < T128, (M, N, K, form)


@pytest.mark.parametrize("M,N,K", [(64, 1280, 23040), (128, 1280, 23040), (256, 1280, 23040), (64, 640, 17280), (80, 800, 21312), (160, 640, 22464)])
@pytest.mark.parametrize("form", [CONV, HALF])
def test_deep_layers_of_few_tiles_stay_in_slices(M, N, K, form):
    """3 x 3 convolutions of the deepest level and other layers whose whole grid of 64 x 80 tiles is a fraction of a round: as many workgroups as
    tiles would walk all of K, where 11 to 22 slices fill the compute units."""
    assert tile_of(M, N, K, form) < T128
    assert tile_of(128, 1280, 32768, form) < T128 and tile_of(128, 1280, 32768, LINEAR) < T128


def test_many_rounds_and_whole_rounds_of_larger_tiles_keep_them():
    for M, N, K in [(49284, 1280, 1504), (73728, 1120, 1440), (60236, 960, 1760), (86640, 1280, 1440)]:
        assert tile_of(M, N, K, HALF) < T128
    for M, N, K in [(1024, 3840, 1280), (16384, 320, 1280), (4096, 1280, 1280), (512, 10240, 1280)]:
        assert tile_of(M, N, K, HALF) < T128
    assert tile_of(32768, 320, 8640, CONV) < T128 and tile_of(32768, 320, 5760, CONV) < T128
    assert tile_of(8192, 1280, 11520, CONV) < T128 and tile_of(8192, 640, 11520, CONV) == T128


def test_linear_layers_of_deep_k_or_several_rounds_keep_their_plans():
    """In the hardware's encodings, where the other kernels are sure to be as fast or the model is not sure enough: more than one round of the tiles,
    codes beyond the caches; convolutions of more than two rounds, and of K up to 128, likewise."""
    for M, N, K in [(3090, 2458, 24304), (31659, 219, 8224), (1724, 2288, 9552), (2230, 1651, 4208), (4960, 1361, 4736), (281, 9415, 3472),
                    (10521, 995, 30672), (5215, 322, 15184), (3834, 392, 29888), (4109, 71, 13984), (1901, 343, 23168), (2890, 184, 29184)]:
        assert tile_of(M, N, K, LINEAR) < T128, (M, N, K)
    for M, N, K in [(9120, 814, 10800), (7986, 999, 7920), (175, 730, 32), (936, 230, 48), (1140, 99, 32), (4270, 199, 128)]:
        assert tile_of(M, N, K, CONV) < T128, (M, N, K)
    # what the tiles are for stays with them
    for M, N, K in [(1290, 939, 11152), (767, 3078, 9280), (542, 2514, 3344), (626, 7481, 3904)]:
        assert tile_of(M, N, K, LINEAR) >= T128, (M, N, K)


def check_tile(rule, query, tile):
    """tile 0: any other kernel."""
    assert rule == tile or (tile == 0 and rule < T128), "this shape no longer takes the tile it is here to cover"
    assert (query if query[0] in KERNEL.values() else 0) == ((KERNEL[tile], 1) if tile else 0), "the query names another kernel"


KERNEL = {T128: B.FPQ_KERNEL_128x80, T64: B.FPQ_KERNEL_64x80}
# M, K, N, tile
LINEAR_CASES = [(2048, 4096, 1280, T128), (2047, 1584, 1279, T128), (1407, 4544, 641, T64), (3000, 3632, 641, T128), (2049, 4640, 321, T64)]


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw", FORMS)
@pytest.mark.parametrize("M,K,N,tile", LINEAR_CASES)
def test_linear(M, K, N, tile, fx, fw):
    print(M, K, N, fx, fw, flush=True)
    if fx == E4M3:
        assert tile_of(M, N, K, LINEAR) == tile, "this shape no longer takes the tile it is here to cover"
    x = synth.activations((M, K), 400 + M)
    w = synth.weights((N, K), 500 + N)
    bias = np.linspace(-1, 1, N).astype(np.float32) if N % 2 else None
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, None)
    rows = np.unique(np.concatenate([np.arange(70), np.arange(M - 140, M), np.random.default_rng(M).integers(0, M, 60)]))
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias, rows=rows)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    buf = torch.full((M * N + 8,), float("nan"), dtype=torch.float32, device=DEV)
    y = buf[4:4 + M * N].view(M, N)
    ws = torch.empty(max(256, B.fpq_gemm_workspace_size(M, N, K, 0)), dtype=torch.uint8, device=DEV)

    def run(flag):
        B.fpq_gemm(dev(xq), 0, fx, sx, None, packed, fw, sw_t, None if bias is None else dev(bias), y, M, N, K, flag, ws)
        torch.cuda.synchronize()

    run(0)
    once = y.cpu().numpy().copy()
    assert not np.isnan(once).any(), "unwritten outputs"
    check_close(once[rows], Y, T, what="linear")
    y.fill_(1.0)
    run(B.FPQ_OUT_ACCUMULATE)
    h = buf.cpu().numpy()
    assert np.isnan(h[:4]).all() and np.isnan(h[-4:]).all(), "written outside the result"
    assert np.allclose(h[4:-4].reshape(M, N), once + np.float32(1), rtol=1e-6, atol=1e-6 * np.abs(once).max())


# B, Cin, H, W, Cout, kernel, stride, padding, tile
CONV_CASES = [(8, 256, 16, 16, 1280, 3, 1, 1, T128), (3, 200, 75, 53, 392, 3, 2, 1, T64), (5, 33, 37, 57, 79, 3, 1, 0, T64),
              (2, 640, 33, 31, 80, 1, 1, 0, T64), (6, 48, 25, 61, 239, 5, 1, 2, T128), (7, 20, 59, 35, 79, 5, 2, 2, T64),
              (300, 384, 3, 1, 640, 3, 1, 1, T64), (2, 20, 21, 45, 321, 5, 2, 3, T64), (4, 33, 36, 47, 321, 3, 1, 0, T128)]


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw", FORMS)
@pytest.mark.parametrize("case", CONV_CASES)
def test_conv(case, fx, fw):
    print(case, fx, fw, flush=True)
    Bn, Cin, H, W, Cout, k, stride, pad, tile = case
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    M = Bn * Ho * Wo
    if fx == E4M3:
        assert tile_of(M, Cout, k * k * B.fpq_padded_channels(Cin), CONV, Ho * Wo % 4 != 0) == tile, \
            "this shape no longer takes the tile it is here to cover"
    x = synth.activations((Bn, Cin, H, W), 600 + Cin)
    w = synth.weights((Cout, Cin, k, k), 700 + Cout)
    bias = np.linspace(-0.5, 0.5, Cout).astype(np.float32) if Cout % 4 else None
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, None)
    pos = np.unique(np.concatenate([np.arange(min(M, 70)), np.arange(max(0, M - 140), M), np.random.default_rng(M).integers(0, M, 60)]))
    Y, T = oracle.conv2d(xq, fx, sx, wq, fw, sw, bias, stride=stride, pad=pad, pix=pos)
    packed, sw_t, _ = gpu_pack(w, fw, None, want_codes=False)
    codes = torch.empty(Bn * H * W * B.fpq_padded_channels(Cin), dtype=torch.uint8, device=DEV)
    B.fpq_quantize_nhwc(dev(x), fx, sx, None, codes)
    buf = torch.full((M * Cout + 8,), float("nan"), dtype=torch.float32, device=DEV)
    y = buf[4:4 + M * Cout]
    ws = torch.empty(max(256, B.fpq_conv2d_workspace_size(Bn, Cin, H, W, Cout, k, k, stride, pad, 0)), dtype=torch.uint8, device=DEV)

    def run(flag):
        B.fpq_conv2d(codes, 0, fx, sx, None, packed, fw, sw_t, None if bias is None else dev(bias), y, Bn, Cin, H, W, Cout, k, k, stride,
                     pad, flag, ws)
        torch.cuda.synchronize()

    run(0)
    once = y.cpu().numpy().copy()
    assert not np.isnan(once).any(), "unwritten outputs"
    check_close(once.reshape(Bn, Cout, Ho * Wo)[pos // (Ho * Wo), :, pos % (Ho * Wo)], Y, T, what="conv")
    y.fill_(1.0)
    run(B.FPQ_OUT_ACCUMULATE)
    h = buf.cpu().numpy()
    assert np.isnan(h[:4]).all() and np.isnan(h[-4:]).all(), "written outside the result"
    assert np.allclose(h[4:-4], once + np.float32(1), rtol=1e-6, atol=1e-6 * np.abs(once).max())


# The tile of each shape above where both operands are moved into halves (0: any other kernel)
LINEAR_HALVES = [T128, T128, 0, T128, 0]
CONV_HALVES = [T128, T64, T64, T64, T128, T64, T64, T64, T128]
# Further shapes, with both tiles: linear layers that take 64 x 80 as halves too
MORE_LINEAR = [(1033, 4016, 1039, T64, T64), (457, 1216, 2387, T64, T64)]
MORE_CONV = [  # three steps for four wavefronts
    (2, 5, 53, 81, 10, 3, 1, 1, T64, T64), (1, 192, 19, 21, 199, 1, 1, 1, T64, T64), (5, 176, 20, 31, 61, 1, 2, 0, T64, T64),
    # fewer rows than a tile has, and fewer columns
    (1, 640, 8, 8, 1280, 3, 2, 1, T64, 0), (1, 33, 5, 9, 7001, 3, 1, 1, T64, T64), (1, 16, 7, 7, 1, 3, 1, 1, T64, T64)]


@pytest.mark.parametrize("fx,fw", FORMS)
def test_tile_of_every_shape_and_operand_pair(fx, fw):
    hardware = fx == E4M3
    for M, K, N, tile, half in [c + (h,) for c, h in zip(LINEAR_CASES, LINEAR_HALVES)] + MORE_LINEAR:
        check_tile(tile_of(M, N, K, LINEAR if hardware else HALF), B.fpq_gemm_launch_plan(M, N, K, fx, fw), tile if hardware else half)
    for Bn, Cin, H, W, Cout, k, stride, pad, tile, half in [c + (h,) for c, h in zip(CONV_CASES, CONV_HALVES)] + MORE_CONV:
        Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
        rule = tile_of(Bn * Ho * Wo, Cout, k * k * B.fpq_padded_channels(Cin), CONV if hardware else HALF, Ho * Wo % 4 != 0)
        check_tile(rule, B.fpq_conv2d_launch_plan(Bn, Cin, H, W, Cout, k, k, stride, pad, fx, fw), tile if hardware else half)


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw", FORMS)
@pytest.mark.parametrize("M,K,N,tile,half", MORE_LINEAR)
def test_linear_in_halves_too(M, K, N, tile, half, fx, fw):
    test_linear(M, K, N, tile, fx, fw)


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw", FORMS)
@pytest.mark.parametrize("case", MORE_CONV)
def test_conv_of_few_steps_rows_and_columns(case, fx, fw):
    test_conv(case[:9], fx, fw)
