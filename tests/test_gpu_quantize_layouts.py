"""Channels-last quantizer and padded rows at the edges of their patches, against the oracle, byte for byte: planes that are no
multiple of four pixels or end with the tensor, channels that fill no group or patch, inputs off 16-byte alignment, and the
formats with and without a conversion instruction; with a scale that is given and one that the layer finds."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 3), (2, 1, 3, 5), (1, 2, 1, 2), (3, 3, 1, 3), (2, 5, 1, 1), (7, 17, 1, 1), (600, 33, 1, 1), (1, 15, 7, 9),
          (2, 16, 8, 8), (3, 66, 5, 13), (2, 64, 9, 7), (5, 130, 2, 2), (1, 200, 13, 53), (66000, 2, 1, 2),
          # patches of 16 and 32 channels, from 513 of 64 pixels on: several images of up to 64 pixels side by side, planes of one patch
          # and one pixel more
          (514, 3, 8, 8), (515, 16, 7, 9), (513, 1, 8, 8), (260, 1, 5, 13), (513, 17, 8, 8), (514, 32, 7, 9), (130, 4, 16, 16), (150, 3, 1, 257),
          (257, 20, 8, 16), (172, 32, 3, 43), (512, 3, 8, 8), (512, 32, 8, 8), (263000, 2, 1, 2), (132000, 17, 1, 2), (66000, 33, 1, 2)]


def padded(codes, C):
    out = np.zeros(codes.shape[:-1] + (B.fpq_padded_channels(C),), dtype=np.uint8)
    out[..., :C] = codes
    return out


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("fmt", [synth.E4M3, synth.E5M2, synth.E3M4])
@pytest.mark.parametrize("off", [0, 1, 2])
def test_channels_last_codes(shape, fmt, off):
    n = int(np.prod(shape))
    x = synth.activations((n + off,), n + off)
    scale = float(np.float32(0.0371))
    want = padded(oracle.quantize(x[off:], fmt, scale).reshape(shape).transpose(0, 2, 3, 1), shape[1])
    codes = torch.full((want.size + 16,), 0xEE, dtype=torch.uint8, device=DEV)
    B.fpq_quantize_nhwc(dev(x)[off:].view(shape), fmt, scale, None, codes)
    torch.cuda.synchronize()
    got = codes.cpu().numpy()
    assert np.array_equal(got[:want.size].reshape(want.shape), want)
    assert np.all(got[want.size:] == 0xEE)


def test_padding_of_any_scale_is_code_zero():
    """Codes of padding channels do not depend on the scale, not even on one that makes every product NaN."""
    for shape in [(3, 5, 4, 4), (9, 5, 1, 1)]:
        codes = torch.empty(shape[0] * shape[2] * shape[3] * 16, dtype=torch.uint8, device=DEV)
        B.fpq_quantize_nhwc(torch.zeros(shape, device=DEV), synth.E4M3, 0.0, torch.zeros(1, device=DEV), codes)
        torch.cuda.synchronize()
        assert np.all(codes.cpu().numpy().reshape(-1, 16)[:, 5:] == 0)


@pytest.mark.parametrize("M,K", [(17, 1), (40, 7), (333, 101), (2000, 1001), (19, 66)])
def test_rows_with_a_scale_found_by_the_layer(M, K):
    """A dynamic-scale layer leaves its codes at the start of its workspace: M rows of K codes, padded to 16."""
    x, w = synth.activations((M, K), M), synth.weights((24, K), K)
    sx = oracle.scale_from_absmax(oracle.absmax(x), synth.E4M3[3])
    packed = torch.empty(B.fpq_packed_size(24, K, 1, 1, synth.E4M3), dtype=torch.uint8, device=DEV)
    sw, y = torch.empty(24, device=DEV), torch.empty((M, 24), device=DEV)
    B.fpq_pack_weights(dev(w), synth.E4M3, None, None, packed, sw)
    ws = torch.empty(B.fpq_gemm_workspace_size(M, 24, K, B.FPQ_X_FP32_DYNAMIC), dtype=torch.uint8, device=DEV)
    B.fpq_gemm(dev(x), B.FPQ_X_FP32_DYNAMIC, synth.E4M3, 0.0, None, packed, synth.E4M3, sw, None, y, M, 24, K, B.FPQ_ACC_FP32, ws)
    torch.cuda.synchronize()
    want = padded(oracle.quantize(x, synth.E4M3, sx), K)
    assert np.array_equal(ws.cpu().numpy()[:want.size].reshape(want.shape), want)


@pytest.mark.parametrize("n", [5, 4096 * 3 + 2, (9 << 20) - 3, 9 << 20, (9 << 20) + 1026, (16 << 20) - 1, (16 << 20) + 4099])
@pytest.mark.parametrize("fmt", [synth.E4M3, synth.E5M2, synth.E3M4, synth.E2M1])
def test_flat_codes_of_a_given_scale(n, fmt):
    """Either side of the sizes at which the kernel changes, in shares that end inside a round; host and device scale."""
    x = synth.activations((n,), n)
    scale = float(np.float32(0.0371))
    want = oracle.quantize(x, fmt, scale)
    if 1 + fmt[0] + fmt[1] <= 4:
        pairs = np.concatenate([want, np.zeros(n % 2, dtype=np.uint8)])
        want = pairs[0::2] | (pairs[1::2] << 4)
    for dev_scale in (None, dev(np.array([scale], dtype=np.float32))):
        codes = torch.full((want.size + 16,), 0xEE, dtype=torch.uint8, device=DEV)
        B.fpq_quantize(dev(x), fmt, 0.0 if dev_scale is not None else scale, dev_scale, codes)
        torch.cuda.synchronize()
        got = codes.cpu().numpy()
        assert np.array_equal(got[:want.size], want) and np.all(got[want.size:] == 0xEE)
