"""The kernel that keeps the weights of a short K in registers (a K of at most 320 codes, every output from one row of
activations), at its edges, against the oracle: every number of 64-code steps, rows and columns that fill no block or
strip, images that end inside a block, output rows that share cache lines, and results as codes."""
import os
import subprocess

import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, dev, gpu_pack
from test_gpu_codes_out import test_linear_activation_then_codes as linear_activation_case
from test_gpu_codes_out import test_conv_silu_then_codes as conv_silu_case
from test_gpu_tiles import FORMS
from test_gpu_tiles import test_conv as conv_case
from test_gpu_tiles import test_linear as linear_case

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2408_06995_amd", "csrc")
E4M3, E2M1, E3M4 = synth.E4M3, synth.E2M1, synth.E3M4

# results in rows: from 144 pairs of 128 rows and 64 columns on; 16 .. 320 codes, all remainders of the 64-code steps' chunks.  The first
# one leaves three of four wavefronts without a block, at the largest K.
LINEAR = [(17, 320, 9216), (33, 64, 9217), (450, 80, 9248), (1001, 128, 4640), (2311, 144, 512), (3000, 192, 448),
          (4640, 208, 200), (9217, 256, 65), (9300, 272, 127), (18500, 304, 64), (4700, 320, 256), (18433, 16, 96),
          (70000, 320, 64)]


def test_the_shapes_take_the_kernel(tmp_path):
    """All forms of every shape of LINEAR, and the lines of the rule for short K."""
    want = [(M, N, K, hw, four, 1) for M, K, N in LINEAR for hw, four in ((1, 0), (1, 1), (0, 0), (0, 1))]
    want += [(2960, 1398, 112, 1, 1, 0), (20551, 2208, 64, 1, 1, 0), (20551, 2208, 64, 1, 0, 1), (1851, 1152, 112, 1, 0, 0),
             (1851, 1152, 112, 0, 0, 1), (500, 1000, 256, 1, 0, 0), (33000, 1001, 320, 1, 0, 0), (33000, 1001, 256, 1, 0, 1)]
    src, out = str(tmp_path / "rule.cpp"), str(tmp_path / "rule")
    with open(src, "w") as f:
        f.write('#include "strip_rule.h"\n#include <stdio.h>\nint main() { int bad = 0;\n')
        for M, N, K, hw, four, yes in want:
            f.write('if (fpq::strip_rows(%d, %d, %d, %d, %d) != %d) bad = printf("%d x %d -> %d, %d %d\\n");\n' %
                    (M, N, K, hw, four, yes, M, K, N, hw, four))
        f.write("return bad != 0; }\n")
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-I", CSRC, src, "-o", out])
    assert subprocess.run([out], capture_output=True, text=True).stdout == ""


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("M,K,N", LINEAR)
def test_rows(M, K, N, fx, fw, acc):
    linear_case(M, K, N, fx, fw, acc)


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("case", [(1, 320, 5, 5, 32, 1, 1, 0), (3, 64, 9, 7, 64, 1, 1, 0), (2, 100, 16, 16, 65, 1, 1, 0),
                                  (5, 3, 11, 13, 130, 1, 1, 0), (2, 160, 64, 32, 320, 1, 1, 0), (9, 250, 33, 31, 72, 1, 1, 0),
                                  (4, 300, 32, 64, 127, 1, 1, 0), (40, 20, 3, 3, 100, 1, 1, 0), (17, 48, 1, 1, 40, 1, 1, 0)])
def test_nchw(case, fx, fw, acc):
    conv_case(case, fx, fw, acc)


@pytest.mark.gpu
@pytest.mark.parametrize("fw,fy,acc", [(E4M3, E4M3, 0), (E2M1, E4M3, 0), (E4M3, E3M4, 0), (E4M3, E4M3, 1), (E2M1, E4M3, 1)])
@pytest.mark.parametrize("act", ["silu", "geglu"])
@pytest.mark.parametrize("M,K,N", [(17, 320, 32), (33, 64, 96), (100, 80, 2560), (1500, 192, 160), (4097, 256, 64), (3000, 304, 544)])
def test_linear_codes_out(M, K, N, fw, fy, acc, act):
    linear_activation_case(M, K, N, fw, fy, acc, act)


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2, 128, 5, 5, 36, 1, 1, 0), (1, 320, 15, 7, 66, 1, 1, 0), (2, 20, 31, 33, 130, 1, 1, 0),
                                  (3, 200, 20, 20, 16, 1, 1, 0), (2, 256, 32, 32, 320, 1, 1, 0)])
def test_conv_codes_out(case):
    conv_silu_case(case)


def _codes_and_weights(M, K, N, fx, fw, seed):
    x = synth.activations((M, K), seed)
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    packed, sw_t, _ = gpu_pack(synth.weights((N, K), seed + 1), fw, None, want_codes=False)
    return dev(oracle.quantize(x, fx, sx)), dev(np.array([sx], dtype=np.float32)), packed, sw_t


@pytest.mark.gpu
@pytest.mark.parametrize("fx,fw,acc", FORMS)
@pytest.mark.parametrize("M,K,N", [(4700, 320, 256), (9300, 272, 127), (2311, 144, 512), (18500, 64, 64)])
def test_single_calls_have_the_bits_of_grouped_ones(M, K, N, fx, fw, acc):
    """The same sums in the same order as on the 64 x 64 tile of the grouped call."""
    xq, sx, packed, sw_t = _codes_and_weights(M, K, N, fx, fw, 1000 + K)
    bias = dev(np.linspace(-1, 1, N).astype(np.float32))
    one, group = torch.full((M, N), float("nan"), device=DEV), torch.full((M, N), float("nan"), device=DEV)
    B.fpq_gemm(xq, 0, fx, 0.0, sx, packed, fw, sw_t, bias, one, M, N, K, acc, None)
    B.fpq_gemm_grouped(B.gemm_problems([(xq, sx, packed, sw_t, bias, group, M, N, K)]), B.FPQ_X_CODES, fx, fw, acc, None)
    torch.cuda.synchronize()
    assert torch.equal(one, group)


@pytest.mark.gpu
@pytest.mark.parametrize("fw", [E4M3, E2M1])
@pytest.mark.parametrize("form", ["rows", "nchw", "codes"])
@pytest.mark.parametrize("M,K,N", [(4700, 320, 256), (9300, 272, 127), (9217, 48, 65)])
def test_scales_and_bias_off_16_byte_alignment(M, K, N, form, fw):
    """sw and bias are fetched sixteen bytes at a time: from an address that is a multiple of four, and up to their last element, which
    may be the last of its buffer."""
    xq, sx, packed, sw_t = _codes_and_weights(M, K, N, E4M3, fw, 1100 + K)
    bias_t = dev(np.linspace(-1, 1, N).astype(np.float32))
    got = []
    for off in (0, 1, 2, 3):
        sw, bias = torch.full((off + N,), float("nan"), device=DEV), torch.full((off + N,), float("nan"), device=DEV)
        sw[off:], bias[off:] = sw_t, bias_t
        y = torch.full((M * N,), float("nan"), device=DEV)
        q = torch.full((M * B.fpq_padded_channels(N),), 0xEE, dtype=torch.uint8, device=DEV)
        if form == "rows":
            B.fpq_gemm(xq, 0, E4M3, 0.0, sx, packed, fw, sw[off:], bias[off:], y, M, N, K, 0, None)
        elif form == "nchw":
            B.fpq_conv2d(xq, 0, E4M3, 0.0, sx, packed, fw, sw[off:], bias[off:], y, 1, K, 1, M, N, 1, 1, 1, 0, 0, None)
        else:
            B.fpq_gemm_codes_out(xq, 0, E4M3, 0.0, sx, packed, fw, sw[off:], bias[off:], E4M3, 0.01, None, q, M, N, K, 0, None)
        torch.cuda.synchronize()
        got.append((y.cpu().numpy(), q.cpu().numpy()))
        assert form == "codes" or not np.isnan(got[-1][0]).any()
    for y, q in got[1:]:
        assert np.array_equal(y, got[0][0], equal_nan=True) and np.array_equal(q, got[0][1])
