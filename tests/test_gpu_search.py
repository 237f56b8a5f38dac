"""Encoding / bias search (Section V-A, Algorithm 1): the HIP reduction against the oracle's 444 quantizer passes."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import oracle
from paper_2408_06995_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FP8 = [(2, 5), (3, 4), (4, 3), (5, 2)]
FP4 = [(1, 2), (2, 1)]
# per-candidate error: one fp32 rounding of each difference (2^-24), fp32 sums of <= 512 non-negative terms per
# wavefront and round (<= 512 * 2^-24 relative), fp32 adds across rounds and waves, fp64 across blocks
REL = 1e-4


def run_search(x, encodings, J):
    from paper_2408_06995_amd import binding as B
    xd = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    mse = torch.full((len(encodings) * J,), float("nan"), dtype=torch.float32, device="cuda")
    res = torch.zeros(40, dtype=torch.uint8, device="cuda")
    ws = torch.empty(B.fpq_search_workspace_size(x.size, len(encodings), J), dtype=torch.uint8, device="cuda")
    B.fpq_search_format(xd, encodings, J, mse, res, ws)
    torch.cuda.synchronize()
    return mse.cpu().numpy().reshape(len(encodings), J), B.search_result(res)


def check(x, encodings, J):
    got, r = run_search(x, encodings, J)
    want, best = oracle.search(x, encodings, J)
    assert np.all(np.abs(got - want) <= REL * want + 1e-30), float(np.max(np.abs(got - want) / (want + 1e-30)))
    # the argmin is a floating-point decision: the chosen candidate must be a minimum up to the error bound
    assert want[r.encoding, r.bias_index] <= want.min() * (1 + 2 * REL)
    if want.size > 1 and want[best] * (1 + 2 * REL) < np.partition(want.reshape(-1), 1)[1]:   # unique beyond the bound
        assert (r.encoding, r.bias_index) == best
    e, m = encodings[r.encoding]
    assert (r.ebits, r.mbits, r.int_bias) == (e, m, 1 << (e - 1))
    absmax = oracle.absmax(x)
    cj = oracle.search_candidate(absmax, r.bias_index, J)
    assert r.maxval == np.float32(cj) and r.scale == np.float32(oracle.search_scale(e, m, cj))
    assert abs(r.mse - want[r.encoding, r.bias_index]) <= REL * want[r.encoding, r.bias_index] + 1e-30
    # Eq. (7) at the reported real-valued bias gives back the max value
    assert abs((2 - 2.0 ** -m) * 2.0 ** (2 ** e - r.real_bias - 1) - cj) <= 1e-5 * cj
    return r


@pytest.mark.parametrize("encodings,J", [(FP8, 111), (FP4, 111), (FP8, 7), ([(4, 3)], 1), (FP8 + FP4, 128)])
@pytest.mark.parametrize("n", [1, 5, 2047, 2048, 40000])
def test_search_matches_oracle_small(encodings, J, n):
    check(synth.activations((n,), 300 + n), encodings, J)


def test_search_activation_and_weight_tensors():
    check(synth.activations((1, 320, 64, 64), 2000).reshape(-1), FP8, 111)      # configuration 2's activations
    check(synth.weights((320, 320, 3, 3), 2500).reshape(-1), FP4, 111)          # and weights
    # ragged length and a pointer that is not 16-byte aligned
    xd = torch.from_numpy(np.ascontiguousarray(synth.activations(((1 << 20) + 4,), 9))).cuda()[1:]
    from paper_2408_06995_amd import binding as B
    mse = torch.empty(4 * 111, dtype=torch.float32, device="cuda")
    res = torch.zeros(40, dtype=torch.uint8, device="cuda")
    ws = torch.empty(B.fpq_search_workspace_size(xd.numel(), 4, 111), dtype=torch.uint8, device="cuda")
    B.fpq_search_format(xd, FP8, 111, mse, res, ws)
    torch.cuda.synchronize()
    want, _ = oracle.search(xd.cpu().numpy(), FP8, 111)
    assert np.all(np.abs(mse.cpu().numpy().reshape(4, 111) - want) <= REL * want)


def test_search_degenerate_tensors():
    r = check(np.zeros(1000, np.float32), FP8, 111)
    assert (r.encoding, r.bias_index, r.mse) == (0, 0, 0.0)
    s = np.float32(0.37)
    x = (np.array([0, .5, 1, 1.5, 2, 3, 4, 6] * 50, np.float32) * s * np.tile([1, -1], 200)).astype(np.float32)
    r = check(x, FP4, 111)
    assert (r.encoding, r.bias_index, r.mse) == (1, 110, 0.0)       # the grid the data lies on, found exactly


def test_search_result_feeds_the_quantizer():
    """The (format, scale) the search reports, given to fpq_quantize, reproduces the candidate's error."""
    from paper_2408_06995_amd import binding as B
    x = synth.activations((50000,), 4)
    r = check(x, FP8, 111)
    fmt = (r.ebits, r.mbits, r.int_bias, 0.0)
    xd = torch.from_numpy(x).cuda()
    codes = torch.empty(x.size, dtype=torch.uint8, device="cuda")
    B.fpq_quantize(xd, fmt, r.scale, None, codes)
    deq = torch.empty(x.size, dtype=torch.float32, device="cuda")
    B.fpq_dequantize(codes, fmt, r.scale, deq)
    torch.cuda.synchronize()
    err = np.mean((x.astype(np.float64) - deq.cpu().numpy().astype(np.float64)) ** 2)
    assert abs(err - r.mse) <= 1e-4 * r.mse


def _outliers_and_tiny(n):
    """One huge value, so that most of the tensor lies tens of binades below the maximum, and values down to subnormals."""
    x = synth.activations((n,), 12)
    x[::7] *= np.float32(1e-3)
    x[5::1000] *= np.float32(1e-12)
    x[9::5000] = np.float32(1e-40)
    x[3] = np.float32(1e9)
    return x


BINNED = 480000   # from here on (at 444 candidates) the errors come from interval moments


@pytest.mark.parametrize("n", [BINNED - 1, BINNED, (1 << 19) + 3])
@pytest.mark.parametrize("encodings", [FP8, FP8 + FP4])
def test_search_large_tensors_match_oracle(n, encodings):
    check(synth.activations((n,), 77), encodings, 111)


def test_search_large_tensors_of_unusual_values():
    check(_outliers_and_tiny(BINNED + 1), FP8, 111)
    wide = np.exp(np.random.default_rng(1).uniform(-70, 5, BINNED)).astype(np.float32)
    check(wide, FP8 + [(6, 1)], 111)                                # spread over a hundred binades
    wide[:] = np.float32(1e-30)
    wide[0] = np.float32(1.0)                                       # all but one value far below every interval
    check(wide, FP8, 111)
    s = np.float32(0.37)
    x = (np.array([0, .5, 1, 1.5, 2, 3, 4, 6] * (BINNED // 4), np.float32) * s).astype(np.float32)
    r = check(x, FP4 + [(3, 0)], 128)
    assert (r.encoding, r.bias_index, r.mse) == (1, 127, 0.0)       # exactly zero, as with the direct evaluation
    r = check(np.zeros(BINNED, np.float32), FP8, 111)
    assert (r.encoding, r.bias_index, r.mse) == (0, 0, 0.0)


def _time(xd, encodings, J):
    from paper_2408_06995_amd import binding as B
    mse = torch.empty(len(encodings) * J, dtype=torch.float32, device="cuda")
    res = torch.zeros(40, dtype=torch.uint8, device="cuda")
    ws = torch.empty(B.fpq_search_workspace_size(xd.numel(), len(encodings), J), dtype=torch.uint8, device="cuda")
    t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for i in range(3):
        if i == 1:
            t[0].record()
        B.fpq_search_format(xd, encodings, J, mse, res, ws)
    t[1].record()
    torch.cuda.synchronize()
    return t[0].elapsed_time(t[1]) / 2


@pytest.mark.parametrize("offset", [0, 1])
def test_search_with_an_outlier_is_no_cliff(offset):
    """One value 2^60 times the rest of a large tensor: no element lies in an interval, every one is evaluated directly.
    That may cost what direct evaluation costs (some ten times the ordinary search), not a walk of the whole tensor by a
    few workgroups (hundreds of times)."""
    n = 1 << 22
    x = synth.activations((n + offset,), 31)
    ordinary = _time(torch.from_numpy(x).cuda()[offset:], FP8, 111)
    x[offset + 77] = np.float32(2.0 ** 60)
    xd = torch.from_numpy(x).cuda()[offset:]
    assert _time(xd, FP8, 111) < 40 * ordinary
    # the same values, few enough per call for the oracle, a workgroup's share at a time
    part = np.concatenate([x[offset:offset + (1 << 19) + 5]])
    check(part, FP8 + [(6, 1)], 111)


@pytest.mark.parametrize("k", [-62, -54, -20, 40])
def test_search_scales_with_the_tensor(k):
    """A power of two times the tensor has the same candidates and 4^k times their errors, also where the errors of single
    elements are far outside the range of a float (at 2^-62 the mean errors, which are reported as floats, have 16 bits left)."""
    x = synth.activations((BINNED + 3,), 55)
    want, r0 = run_search(x, FP8 + FP4, 111)
    got, r = run_search(np.ldexp(x, k), FP8 + FP4, 111)
    assert np.all(np.abs(np.ldexp(got.astype(np.float64), -2 * k) - want) <= 1e-6 * want + np.ldexp(1.0, -149 - 2 * k))
    assert (r.encoding, r.bias_index) == (r0.encoding, r0.bias_index)


@pytest.mark.parametrize("offset,outlier", [(0, 0), (1, 0), (0, 60)])
def test_search_has_the_same_bits_every_time(offset, outlier):
    """Repeated calls agree in every bit, and an encoding listed twice has equal errors, of which the first is chosen."""
    x = synth.activations((BINNED + 50001,), 91)
    if outlier:
        x[::3] *= np.float32(2.0 ** -40)
        x[4] = np.float32(2.0 ** (outlier // 4))
    x = x[offset:]
    encodings = [(4, 3), (3, 4), (4, 3), (3, 4), (2, 5), (2, 5), (5, 2), (5, 2)]
    first, r = run_search(x, encodings, 111)
    for _ in range(4):
        again, ra = run_search(x, encodings, 111)
        assert np.array_equal(again, first)
        assert (ra.encoding, ra.bias_index, ra.mse) == (r.encoding, r.bias_index, r.mse)
    for i, j in ((0, 2), (1, 3), (4, 5), (6, 7)):
        assert np.array_equal(first[i], first[j])
    assert r.encoding in (0, 1, 4, 6)
    # errors are compared as doubles: in any order of additions the smallest of eight equal candidates could be any of them
    for _ in range(4):
        assert run_search(x, [(4, 3)] * 8, 111)[1].encoding == 0
    check(x, encodings[:2] + [(5, 2)], 111)


@pytest.mark.parametrize("n", [1000, 524288])
@pytest.mark.parametrize("bad", [[float("nan")], [float("inf")], [float("nan"), float("-inf")]])
def test_search_without_a_finite_error_takes_the_first_candidate(n, bad):
    """With no finite error nothing is less than the first candidate's, in the direct and the binned form; the error is reported
    as it is."""
    x = synth.activations((n,), 77)
    x[n // 3:n // 3 + len(bad)] = bad
    got, r = run_search(x, FP8, 111)
    assert not np.isfinite(got).any()
    assert (r.encoding, r.bias_index) == (0, 0)
    assert r.mse == got[0, 0] or (np.isnan(r.mse) and np.isnan(got[0, 0]))
