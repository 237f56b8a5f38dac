"""fpq_gemm_noalloc, the entry point for callers that cannot allocate device memory: same kernels as fpq_gemm, scratch
space in a static device array inside the library instead of a caller's workspace.  Its output must equal fpq_gemm's
bit for bit (same launch configuration, same summation order) on consecutive calls that share the array, the second
with a smaller input, and fpq_gemm's output is itself compared with the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, check_close, dev, gpu_pack

pytestmark = pytest.mark.gpu


def both_ways(M, K, N, fw, x_kind, seed):
    fx = synth.E4M3
    x = synth.activations((M, K), seed)
    w = synth.weights((N, K), seed + 1)
    h = synth.rounding_mask((N, K), seed + 2) if fw is synth.E2M1 else None
    bias = np.linspace(-0.2, 0.2, N).astype(np.float32)
    sx = oracle.scale_from_absmax(oracle.absmax(x), fx[3])
    xq = oracle.quantize(x, fx, sx)
    wq, sw = oracle.pack_weights(w, fw, h)
    Y, T = oracle.gemm(xq, fx, sx, wq, fw, sw, bias)
    packed, sw_t, _ = gpu_pack(w, fw, h, want_codes=False)
    x_t = dev(xq) if x_kind == B.FPQ_X_CODES else dev(x)
    sx_arg = 0.0 if x_kind == B.FPQ_X_FP32_DYNAMIC else sx
    need = B.fpq_gemm_workspace_size(M, N, K, x_kind)
    assert 0 < need <= B.FPQ_NOALLOC_SCRATCH_BYTES
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    y_ref = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    B.fpq_gemm(x_t, x_kind, fx, sx_arg, None, packed, fw, sw_t, dev(bias), y_ref, M, N, K, B.FPQ_ACC_FP32, ws)
    y_new = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    B.fpq_gemm_noalloc(x_t, x_kind, fx, sx_arg, None, packed, fw, sw_t, dev(bias), y_new, M, N, K, B.FPQ_ACC_FP32)
    torch.cuda.synchronize()
    check_close(y_ref.cpu().numpy(), Y, T, what="fpq_gemm %s" % ((M, K, N),))
    assert torch.equal(y_ref, y_new), "fpq_gemm_noalloc differs from fpq_gemm at %s" % ((M, K, N),)
    check_close(y_new.cpu().numpy(), Y, T, what="fpq_gemm_noalloc %s" % ((M, K, N),))


def test_noalloc_equals_fpq_gemm_on_two_calls_in_a_row():
    # dynamic scale, and room for K slices (the tiles that run have none): activation codes, partial maxima and the scale
    assert B.fpq_gemm_plan(512, 1280, 5120)[1] > 1
    both_ways(512, 5120, 1280, synth.E4M3, B.FPQ_X_FP32_DYNAMIC, 11)
    # a smaller input right after, which reuses the front of the same array: sliced again, fp32 input with a given scale
    assert B.fpq_gemm_plan(384, 640, 3072)[1] > 1
    both_ways(384, 3072, 640, synth.E2M1, B.FPQ_X_FP32, 21)
    # and one on codes, where only the partial sums live in the scratch
    both_ways(300, 2880, 320, synth.E4M3, B.FPQ_X_CODES, 31)


def test_noalloc_equals_fpq_gemm_in_slices_of_160_wide_tiles():
    """The scratch holds activation codes, partial sums, partial maxima and the scale."""
    assert B.fpq_gemm_launch_plan(512, 1280, 11520, synth.E4M3, synth.E4M3) == (B.FPQ_KERNEL_128x160, 8)
    both_ways(512, 11520, 1280, synth.E4M3, B.FPQ_X_FP32_DYNAMIC, 51)
    both_ways(100, 20480, 640, synth.E2M1, B.FPQ_X_FP32_DYNAMIC, 61)


def test_noalloc_rejects_what_does_not_fit():
    L = B.lib()
    f = B.fmt(synth.E4M3)
    import ctypes as C
    p = C.c_void_p(4096)          # never dereferenced: the size check comes first
    M, K, N = 1 << 20, 4096, 320
    assert B.fpq_gemm_workspace_size(M, N, K, 1) > B.FPQ_NOALLOC_SCRATCH_BYTES
    assert L.fpq_gemm_noalloc(p, 1, f, 1.0, None, p, f, p, None, p, M, N, K, 0, None) == -6


def test_noalloc_takes_in_one_slice_what_fits_without_partial_sums():
    # codes of 40.5 MB and the partial sums of three slices exceed the scratch together, the codes alone do not
    M, K, N = 6912, 6144, 300
    assert B.fpq_gemm_workspace_size(M, N, K, B.FPQ_X_FP32_DYNAMIC) > B.FPQ_NOALLOC_SCRATCH_BYTES > M * K + 8192
    x = synth.activations((M, K), 41)
    w = synth.weights((N, K), 42)
    sx = oracle.scale_from_absmax(oracle.absmax(x), synth.E4M3[3])
    rows = np.r_[0:64, 3450:3470, M - 64:M]
    wq, sw = oracle.pack_weights(w, synth.E4M3)
    Y, T = oracle.gemm(oracle.quantize(np.ascontiguousarray(x[rows]), synth.E4M3, sx), synth.E4M3, sx, wq, synth.E4M3, sw, None)
    packed, sw_t, _ = gpu_pack(w, synth.E4M3, None, want_codes=False)
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    B.fpq_gemm_noalloc(dev(x), B.FPQ_X_FP32_DYNAMIC, synth.E4M3, 0.0, None, packed, synth.E4M3, sw_t, None, y, M, N, K,
                       B.FPQ_ACC_FP32)
    assert not torch.isnan(y).any()
    check_close(y.cpu().numpy()[rows], Y, T, what="fpq_gemm_noalloc in one slice")
