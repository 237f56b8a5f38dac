"""Rounding learning (Section V-B, Eq. (10)-(14)): the HIP step against the double-precision oracle.

Tolerances.  The step is fp32 throughout: the output error R = A (Wq - W)^T is a sum of K products of fp32 values whose
second factor carries the rounding of Wq - W (one ulp of |W|), so |R_gpu - R| <= 1e-5 * sum_k |A_k| (|D_k| + 1e-6 |W_k|);
the losses are sums of non-negative terms (relative 1e-4); the gradient d mse / d Wq is a sum over M rows of products R A
with the error of R carried through, bounded by 2e-5 * (2 / (M N)) sum_m (|R| + err R) |A|, times d Wq / d alpha."""
import numpy as np
import pytest
import torch

import oracle
from oracle import rounding as R
from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth
from gpu_util import DEV, dev

pytestmark = pytest.mark.gpu

E2M1, E4M3, E1M2 = synth.E2M1, synth.E4M3, (1, 2, 1, 1.75)


def layer(N, K, M, seed, fmt):
    W = synth.weights((N, K), seed)
    sw = (np.abs(W).max(axis=1) / np.float32(fmt[3])).astype(np.float32)
    A = synth.activations((M, K), seed + 1)
    rng = np.random.default_rng(seed + 2)
    alpha = rng.normal(0, 2, (N, K)).astype(np.float32)
    return W, sw, A, alpha


def gpu_step(W, sw, alpha, A, fmt, lr, regw, want_grad=True):
    N, K = W.shape
    M = A.shape[0]
    al = dev(alpha.copy())
    loss = torch.full((2,), float("nan"), device=DEV)
    grad = torch.full((N, K), float("nan"), device=DEV) if want_grad else None
    ws = torch.empty(B.fpq_rl_workspace_size(M, N, K), dtype=torch.uint8, device=DEV)
    B.fpq_rl_step(dev(W), dev(sw), fmt, al, dev(A), lr, regw, loss, grad, ws)
    torch.cuda.synchronize()
    return al.cpu().numpy(), loss.cpu().numpy(), None if grad is None else grad.cpu().numpy()


# N, K, M: below one tile, ragged in every direction, several 64-tiles, the 128-tile kernel, a deep contraction over M
SHAPES = [(3, 5, 6), (33, 70, 45), (130, 96, 200), (320, 320, 256), (640, 1280, 2048), (64, 48, 5000)]


@pytest.mark.parametrize("N,K,M", SHAPES)
@pytest.mark.parametrize("fmt", [E2M1, E4M3, E1M2])
def test_step_against_oracle(N, K, M, fmt):
    check_step(N, K, M, fmt, 9000 + N)


@pytest.mark.parametrize("i", range(24))
def test_step_on_random_shapes(i):
    """Shapes drawn at random: every combination of ragged tiles of the two fp32 contractions and of their K slices."""
    rng = np.random.default_rng(9500 + i)
    N, K, M = int(rng.integers(1, 400)), int(rng.integers(1, 500)), int(rng.integers(1, 3000))
    fmt = [E2M1, E4M3, E1M2, (3, 0, 4, 8.0)][i % 4]
    print("case", i, (N, K, M), fmt, flush=True)
    check_step(N, K, M, fmt, 9600 + i)


def check_step(N, K, M, fmt, seed):
    W, sw, A, alpha = layer(N, K, M, seed, fmt)
    lr, regw = 50.0, 0.3
    a1, loss, grad = gpu_step(W, sw, alpha, A, fmt, lr, regw)
    mse, reg = R.loss(W, sw, alpha, A, fmt, regw)
    assert loss[0] == pytest.approx(mse, rel=1e-4)
    assert loss[1] == pytest.approx(reg, rel=1e-4)
    # gradient: bound from the module docstring
    Wq, dWq = R.soft_weights(W, sw, alpha, fmt)
    A64, W64 = A.astype(np.float64), W.astype(np.float64)
    D = Wq - W64
    Rm = A64 @ D.T
    errR = 1e-5 * (np.abs(A64) @ (np.abs(D) + 1e-6 * np.abs(W64)).T)
    errG = 2e-5 * (2.0 / Rm.size) * ((np.abs(Rm) + errR).T @ np.abs(A64)) + (2.0 / Rm.size) * (errR.T @ np.abs(A64))
    g = R.gradient(W, sw, alpha, A, fmt, regw)
    # plus the fp32 evaluation of the two terms themselves (they can cancel in g)
    Gm = (2.0 / Rm.size) * (Rm.T @ A64)
    tol = errG * np.abs(dWq) + 1e-5 * (np.abs(Gm * dWq) + regw * np.abs(R.regulariser(alpha)[1])) + 1e-12
    bad = np.abs(grad - g) > tol
    assert not bad.any(), (int(bad.sum()), float((np.abs(grad - g) / tol).max()))
    # the update is alpha - lr * (the gradient the kernel reports), in fp32
    assert np.allclose(a1, alpha - np.float32(lr) * grad, rtol=1e-6, atol=1e-7)


@pytest.mark.parametrize("fmt", [E2M1, E4M3, (3, 0, 4, 8.0)])
def test_init_alpha_and_mask(fmt):
    N, K = 37, 129
    W = synth.weights((N, K), 9500)
    W[0, :3] = [0.0, -0.0, W[1].max() * 5]
    sw = (np.abs(W[1:]).max() / np.float32(fmt[3]) * np.ones(N)).astype(np.float32)
    al = torch.full((N, K), float("nan"), device=DEV)
    B.fpq_rl_init_alpha(dev(W), dev(sw), fmt, al)
    mk = torch.full((N * K,), 7, dtype=torch.uint8, device=DEV)
    B.fpq_rl_mask(al, mk)
    torch.cuda.synchronize()
    a_gpu = al.cpu().numpy()
    a0 = R.init_alpha(W, sw, fmt)
    assert np.allclose(a_gpu, a0, rtol=1e-5, atol=1e-5)
    assert np.array_equal(mk.cpu().numpy().reshape(N, K), (a_gpu >= 0).astype(np.uint8))
    agree = mk.cpu().numpy().reshape(N, K) == R.mask(a0)
    assert agree.mean() > 0.999                                # only alphas within rounding of 0 may differ
    assert np.all(np.abs(a0[~agree]) < 1e-5)


def test_learning_run_follows_the_oracle_and_feeds_pack_weights():
    """40 steps from the initial alpha on a small layer: the loss curve follows the oracle's, and the learned mask goes
    through fpq_pack_weights like any other mask."""
    fmt = E2M1
    N, K, M = 64, 96, 512
    W, sw, A, _ = layer(N, K, M, 9700, fmt)
    lr, regw = 3000.0, 0.01
    al = torch.empty((N, K), device=DEV)
    Wd, swd, Ad = dev(W), dev(sw), dev(A)
    B.fpq_rl_init_alpha(Wd, swd, fmt, al)
    loss = torch.zeros(2, device=DEV)
    ws = torch.empty(B.fpq_rl_workspace_size(M, N, K), dtype=torch.uint8, device=DEV)
    a_or = R.init_alpha(W, sw, fmt)
    curve_gpu, curve_or = [], []
    for _ in range(40):
        B.fpq_rl_step(Wd, swd, fmt, al, Ad, lr, regw, loss, None, ws)
        curve_gpu.append(loss.cpu().numpy().copy())
        a_or, mse, reg = R.step(W, sw, a_or, A, fmt, lr, regw)
        curve_or.append((mse, reg))
    curve_gpu, curve_or = np.array(curve_gpu), np.array(curve_or)
    assert np.allclose(curve_gpu[:, 1], curve_or[:, 1], rtol=2e-3)
    assert np.allclose(curve_gpu[1:, 0], curve_or[1:, 0], rtol=2e-2)        # the first entry is ~0: start = unquantized weights
    assert curve_gpu[-1, 1] < curve_gpu[0, 1]                               # decisions sharpen
    mk = torch.empty(N * K, dtype=torch.uint8, device=DEV)
    B.fpq_rl_mask(al, mk)
    torch.cuda.synchronize()
    h = mk.cpu().numpy().reshape(N, K)
    from gpu_util import gpu_pack
    _, _, codes = gpu_pack(W, fmt, h, scale_np=sw)
    wq, _ = oracle.pack_weights(W, fmt, h, sw)
    assert np.array_equal(codes, wq)
    # the learned rounding is not worse at the layer output than round-to-nearest (what learning is for)
    A64 = A.astype(np.float64)
    def out_err(cq):
        return float(np.mean((A64 @ (oracle.dequantize(cq, fmt) * sw.astype(np.float64)[:, None] - W.astype(np.float64)).T) ** 2))
    near, _ = oracle.pack_weights(W, fmt, None, sw)
    assert out_err(wq) <= out_err(near) * 1.05


@pytest.mark.parametrize("case", [(2, 5, 9, 7, 3, 1, 1), (1, 16, 12, 12, 3, 2, 1), (3, 4, 6, 6, 1, 1, 0), (1, 3, 11, 8, 5, 1, 2)])
def test_patch_matrix_exact_and_conv_step(case):
    """The patch matrix is a copy (exact); a rounding-learning step of a convolution = the linear step on it."""
    Bn, C, H, W, k, stride, pad = case
    x = synth.activations((Bn, C, H, W), 9800 + C)
    Ho, Wo = (H + 2 * pad - k) // stride + 1, (W + 2 * pad - k) // stride + 1
    M, K = Bn * Ho * Wo, C * k * k
    a = torch.full((M, K), float("nan"), device=DEV)
    B.fpq_rl_im2col(dev(x), k, k, stride, pad, a)
    torch.cuda.synchronize()
    A = R.im2col(x, k, k, stride, pad)
    assert np.array_equal(a.cpu().numpy().astype(np.float64), A)
    fmt = E2M1
    N = 6
    Wt = synth.weights((N, C, k, k), 9850).reshape(N, K)
    sw = (np.abs(Wt).max(axis=1) / np.float32(fmt[3])).astype(np.float32)
    alpha = R.init_alpha(Wt, sw, fmt).astype(np.float32)
    al = dev(alpha.copy())
    loss = torch.zeros(2, device=DEV)
    grad = torch.zeros((N, K), device=DEV)
    ws = torch.empty(B.fpq_rl_workspace_size(M, N, K), dtype=torch.uint8, device=DEV)
    B.fpq_rl_step(dev(Wt), dev(sw), fmt, al, a, 10.0, 0.1, loss, grad, ws)
    torch.cuda.synchronize()
    mse, reg = R.loss(Wt, sw, alpha, A.astype(np.float32), fmt, 0.1)
    g = R.gradient(Wt, sw, alpha, A.astype(np.float32), fmt, 0.1)
    assert loss.cpu().numpy()[0] == pytest.approx(mse, rel=1e-3, abs=1e-12)
    assert loss.cpu().numpy()[1] == pytest.approx(reg, rel=1e-4)
    assert np.allclose(grad.cpu().numpy(), g, rtol=1e-3, atol=1e-6 * np.abs(g).max() + 1e-12)


def test_argument_checks():
    import ctypes as C
    L = B.lib()
    t = torch.zeros(1024, device=DEV)
    P = C.c_void_p(t.data_ptr())
    f = B.fmt(E2M1)
    assert L.fpq_rl_step(P, P, 4, 4, f, P, P, 4, 0.1, 0.1, P, None, P, 16, None) == -6
    assert L.fpq_rl_step(P, P, 4, 4, f, P, P, 0, 0.1, 0.1, P, None, P, 1 << 20, None) == -4
    assert L.fpq_rl_step(P, P, 4, 4, f, None, P, 4, 0.1, 0.1, P, None, P, 1 << 20, None) == -1
    assert L.fpq_rl_step(P, P, 4, 4, f, P, P, 4, float("nan"), 0.1, P, None, P, 1 << 20, None) == -3
    assert L.fpq_rl_step(P, P, 4, 4, B.fmt((2, 1, 1, 5.0)), P, P, 4, 0.1, 0.1, P, None, P, 1 << 20, None) == -2
    assert L.fpq_rl_init_alpha(P, None, 4, 4, f, P, None) == -1
    assert B.fpq_rl_workspace_size(0, 4, 4) == 0


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (5, 3, 2), (16, 64, 16), (17, 65, 15), (33, 128, 48), (130, 67, 129), (257, 129, 66),
                                   (300, 64, 4), (96, 132, 100), (2050, 130, 36)])
def test_step_at_tile_edges(M, N, K):
    """Shapes either side of the tiles (64, 128 rows), of the steps of 16 k and of the loads' four elements, in both products."""
    check_step(N, K, M, E2M1, 9700 + M)


# Products of at least 256 tiles of 128 x 128 (output error: M x N; gradient: N x K times the slices of M), and the loads they
# take: 16 bytes where rows have a multiple of 4 elements, single elements otherwise.
BIG = [((4100, 1028, 20), "output error, 16-byte loads"), ((4099, 1027, 27), "output error, single elements"),
       ((2050, 645, 1283), "gradient, single elements"), ((2052, 644, 1284), "gradient, 16-byte loads")]


@pytest.mark.parametrize("shape,what", BIG)
def test_step_of_128_tiles(shape, what):
    M, N, K = shape
    check_step(N, K, M, E2M1, 9750 + N)


def test_steps_of_both_loads_in_one_process():
    """A kernel's allowance of more than 64 KB of LDS is its own: both forms run, whichever ran first."""
    for M, N, K in [(4100, 1028, 20), (4099, 1027, 27), (4100, 1028, 20)]:
        check_step(N, K, M, E2M1, 9760 + N)


def test_weights_of_a_convolution_are_refused():
    """The step takes weights as a matrix; a four-dimensional tensor is an error of the caller, not its first two sizes."""
    w = torch.zeros((4, 8, 3, 3), dtype=torch.float32, device=DEV)
    sw, loss, a = (torch.ones(n, dtype=torch.float32, device=DEV) for n in (4, 2, 72))
    ws = torch.empty(4096, dtype=torch.uint8, device=DEV)
    with pytest.raises(ValueError):
        B.fpq_rl_step(w, sw, synth.E4M3, w, a, 1e-2, 1e-3, loss, None, ws)
    with pytest.raises(ValueError):
        B.fpq_quantize_nhwc(w.reshape(1, 4, 8, 3, 3), synth.E4M3, 1.0, None, ws)
    with pytest.raises(TypeError):
        B.fpq_gemm(a, B.FPQ_X_FP32, synth.E4M3, 1.0, None, ws, synth.E4M3, sw, None, loss, 1.5, 1, 16, workspace=ws)


@pytest.mark.parametrize("M,N,K", [(70, 33, 40), (4100, 1028, 20), (4099, 1027, 27)])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_activations_that_are_not_finite(M, N, K, bad):
    """An infinite activation makes the outputs of its row, the loss and the gradient infinite, with the signs of the products; a NaN
    makes them NaN.  (Not against R.loss, which subtracts the two outputs: both are infinite.)"""
    W, sw, A, alpha = layer(N, K, M, 9900 + N, E2M1)
    m, k = M // 2, K // 3
    A[m, k] = bad
    _, loss, grad = gpu_step(W, sw, alpha, A, E2M1, 1.0, 0.3)
    Wq, dWq = R.soft_weights(W, sw, alpha, E2M1)
    D = Wq[:, k] - W[:, k].astype(np.float64)
    sure = np.abs(D) > 1e-5 * np.abs(W[:, k])                      # the sign of an error of a few ulps is the rounding's
    assert sure.sum() > N // 2
    with np.errstate(all="ignore"):
        want = (bad * D)[:, None] * A[m].astype(np.float64) * dWq    # what the row adds to d mse / d alpha, up to 2 / (M N)
    got, want = grad[sure], want[sure]
    assert loss[0] == bad or np.isnan(loss[0]) and (np.isnan(bad) or not sure.all())      # an error of 0 times infinity
    assert np.isfinite(loss[1])
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isposinf(got), np.isposinf(want))


def test_activations_near_the_largest_float():
    """Above the largest bf16 number and still finite: the output error of weights around 1e-30 is as well."""
    W, sw, A, alpha = layer(40, 48, 70, 9950, E2M1)
    W, sw = W * np.float32(2.0 ** -100), sw * np.float32(2.0 ** -100)
    A[5, 7] = np.float32(3.395e38)
    _, loss, _ = gpu_step(W, sw, alpha, A, E2M1, 1.0, 0.3)
    mse, _ = R.loss(W, sw, alpha, A, E2M1, 0.3)
    assert loss[0] == pytest.approx(mse, rel=1e-4)
