"""C-ABI checks that need no GPU: the library loads, exports every declared symbol, its host helpers
agree with the paper's closed forms, and argument validation returns the documented codes before
anything is launched."""
import ctypes as C
import os
import re

import pytest

from paper_2408_06995_amd import binding as B
from paper_2408_06995_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "fpq.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(fpq_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = B.lib()
    names = declared_symbols()
    assert len(names) >= 15
    for n in names:
        assert hasattr(L, n), n
    assert sorted(names) == sorted(B.EXPORTS)


def test_format_max_and_check():
    for line in open(os.path.join(ROOT, "tests", "golden", "format_max.txt")):
        if line.strip() and line[0] != "#":
            e, m, b, c = line.split()
            assert B.fpq_format_max(int(e), int(m), int(b)) == float(c)
    assert B.fpq_format_max(0, 3, 1) == 0.0 and B.fpq_format_max(5, 3, 1) == 0.0
    for f in (synth.E4M3, synth.E5M2, synth.E2M1, synth.E1M2, synth.E3M4, synth.E2M5, synth.E3M0, (4, 3, 7, 0.0),
              (4, 3, 7, 480.0), (4, 3, 7, 0.001953125)):
        assert B.fpq_format_check(f) == 0, f
    for f in ((4, 3, 7, 449.0), (4, 3, 7, 512.0), (4, 3, 7, -448.0), (4, 4, 7, 0.0), (0, 3, 1, 0.0), (2, -1, 1, 0.0),
              (4, 3, 65, 0.0), (4, 3, 7, float("nan")), (4, 3, 7, float("inf"))):
        assert B.fpq_format_check(f) == -2, f


def test_bias_to_scale():
    assert B.fpq_bias_to_scale(4, 3, 7.0) == (7, 1.0)
    ib, sc = B.fpq_bias_to_scale(4, 3, 6.5)
    assert ib == 6 and abs(sc - 2.0 ** -0.5) < 1e-7
    # the grid of real bias b equals scale * grid of the integer bias: c(b) = scale * c(int bias)
    for rb in (3.25, 7.9, -1.5):
        ib, sc = B.fpq_bias_to_scale(4, 3, rb)
        c_real = (2 - 2.0 ** -3) * 2.0 ** (16 - rb - 1)
        assert abs(sc * B.fpq_format_max(4, 3, ib) / c_real - 1) < 1e-6


def test_sizes():
    assert B.fpq_code_bytes(10, synth.E4M3) == 10
    assert B.fpq_code_bytes(11, synth.E2M1) == 6
    assert B.fpq_padded_channels(4) == 16 and B.fpq_padded_channels(320) == 320
    assert B.fpq_packed_size(320, 320, 1, 1, synth.E4M3) == 256 + 320 * 384
    assert B.fpq_packed_size(320, 320, 3, 3, synth.E4M3) == 256 + 320 * 2944
    assert B.fpq_packed_size(1280, 1280, 3, 3, synth.E2M1) == 256 + 1280 * 11520 // 2
    assert B.fpq_packed_size(0, 320, 1, 1, synth.E4M3) == 0
    assert B.fpq_absmax_workspace_size(0) == 4 and B.fpq_absmax_workspace_size(10 ** 9) == 4096
    assert B.fpq_gemm_workspace_size(256, 320, 320, 0) == 0
    assert B.fpq_gemm_workspace_size(256, 320, 320, 1) == 256 * 320
    assert B.fpq_conv2d_workspace_size(1, 4, 64, 64, 320, 3, 3, 1, 1, 1) == 64 * 64 * 16


def test_argument_validation_without_gpu():
    L = B.lib()
    f = B.fmt(synth.E4M3)
    bad = B.fmt((4, 3, 7, 449.0))
    bad_fmt = bad
    p = C.c_void_p(4096)          # never dereferenced: every call below fails validation first
    assert L.fpq_quantize(p, 16, bad, 1.0, None, p, None) == -2
    assert L.fpq_quantize(p, 16, f, 0.0, None, p, None) == -3
    assert L.fpq_quantize(p, 16, f, float("nan"), None, p, None) == -3
    assert L.fpq_quantize(p, 16, f, float("inf"), None, p, None) == -3
    assert L.fpq_quantize(None, 16, f, 1.0, None, p, None) == -1
    assert L.fpq_quantize(p, 16, f, 1.0, None, None, None) == -1
    assert L.fpq_quantize(None, 0, f, 1.0, None, None, None) == 0
    assert L.fpq_quantize(C.c_void_p(4098), 16, f, 1.0, None, p, None) == -5
    assert L.fpq_absmax(p, 16, 448.0, None, None, p, 4, None) == -1
    assert L.fpq_absmax(p, 10 ** 6, 448.0, p, p, p, 4, None) == -6
    assert L.fpq_absmax(p, 16, 0.0, p, p, p, 4, None) == -2
    assert L.fpq_quantize_nhwc(p, 0, 4, 8, 8, f, 1.0, None, p, None) == -4
    assert L.fpq_quantize_nhwc(p, 1, 4, 8, 8, f, 1.0, None, C.c_void_p(4100), None) == -5
    assert L.fpq_pack_weights(p, 8, 0, 1, 1, f, None, None, p, 1 << 20, p, None, None) == -4
    assert L.fpq_pack_weights(p, 8, 32, 1, 1, f, None, None, p, 64, p, None, None) == -6
    assert L.fpq_pack_weights(p, 8, 32, 1, 1, f, None, None, None, 1 << 20, p, None, None) == -1
    e2m1 = B.fmt(synth.E2M1)
    # fpq_gemm: shape, null, scale, alignment, workspace, unsupported format pairing
    assert L.fpq_gemm(p, 0, f, 1.0, None, p, f, p, None, p, 8, 8, 0, 0, None, 0, None) == -4
    assert L.fpq_gemm(None, 0, f, 1.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -1
    assert L.fpq_gemm(p, 0, f, -1.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -3
    assert L.fpq_gemm(p, 0, f, 1.0, None, p, f, p, None, p, 8, 8, 24, 0, None, 0, None) == -5
    assert L.fpq_gemm(p, 1, f, 1.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -6
    assert L.fpq_gemm(p, 2, f, 0.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -6   # dynamic scale: no sx needed
    assert L.fpq_gemm(p, 3, f, 1.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -8
    # encoding / bias search: every check below returns before a launch
    import ctypes as CT
    ee, mm = (CT.c_int32 * 2)(4, 5), (CT.c_int32 * 2)(3, 2)
    bad = (CT.c_int32 * 2)(4, 6)
    ev, mv, bv = CT.cast(ee, CT.c_void_p), CT.cast(mm, CT.c_void_p), CT.cast(bad, CT.c_void_p)
    assert L.fpq_search_format(p, 100, ev, mv, 0, 111, None, p, p, 1 << 20, None) == -4
    assert L.fpq_search_format(p, 100, ev, mv, 2, 129, None, p, p, 1 << 20, None) == -4
    assert L.fpq_search_format(p, 100, ev, mv, 2, 111, None, None, p, 1 << 20, None) == -1
    assert L.fpq_search_format(p, 100, ev, bv, 2, 111, None, p, p, 1 << 20, None) == -2
    assert L.fpq_search_format(p, 100, ev, mv, 2, 111, None, p, p, 64, None) == -6
    assert B.fpq_search_workspace_size(5000, 4, 111) == 4096 + 256 + 3 * 444 * 4 + (256 - 3 * 444 * 4 % 256) % 256
    assert B.fpq_search_workspace_size(5000, 9, 111) == 0
    assert B.fpq_gemm_workspace_size(8, 8, 32, 2) == B.fpq_gemm_workspace_size(8, 8, 32, 1) + 4096 + 256
    assert L.fpq_gemm(p, 0, e2m1, 1.0, None, p, f, p, None, p, 8, 8, 32, 0, None, 0, None) == -8
    assert L.fpq_gemm(p, 0, B.fmt(synth.E3M4), 1.0, None, p, f, p, None, p, 8, 8, 32, 1, None, 0, None) == -8
    assert L.fpq_gemm(p, 0, f, 1.0, None, p, f, p, None, p, 8, 8, 32, 7, None, 0, None) == -8
    assert L.fpq_gemm(p, 0, f, 1.0, None, p, f, p, None, p, 0, 8, 32, 0, None, 0, None) == 0
    assert L.fpq_conv2d(p, 0, f, 1.0, None, p, f, p, None, p, 1, 16, 2, 2, 8, 3, 3, 1, 0, 0, None, 0, None) == -4
    assert L.fpq_conv2d(p, 0, f, 1.0, None, p, f, p, None, p, 1, 16, 8, 8, 8, 3, 3, 0, 1, 0, None, 0, None) == -4
    # a contraction longer than fpq_pack_weights can have packed (2^28 codes per output channel)
    assert L.fpq_conv2d(p, 0, f, 1.0, None, p, e2m1, p, None, p, 1, 1 << 20, 1, 1, 1, 48, 48, 1, 24, 0, None, 0, None) == -4
    assert L.fpq_pack_weights(p, 1, 1 << 20, 48, 48, e2m1, None, None, p, 1 << 40, p, None, None) == -4
    # zero count: null, kind, format, workspace, alignment
    assert B.fpq_count_zeros_workspace_size(10 ** 9) == 8192
    assert L.fpq_count_zeros(p, 0, 100, f, None, p, 8192, None) == -1
    assert L.fpq_count_zeros(None, 0, 100, f, p, p, 8192, None) == -1
    assert L.fpq_count_zeros(p, 2, 100, f, p, p, 8192, None) == -8
    assert L.fpq_count_zeros(p, 0, 100, bad_fmt, p, p, 8192, None) == -2
    assert L.fpq_count_zeros(p, 0, 100, f, p, p, 8184, None) == -6
    assert L.fpq_count_zeros(p, 0, 100, f, C.c_void_p(4100), p, 8192, None) == -5
    assert L.fpq_count_zeros(C.c_void_p(4098), 1, 100, f, p, p, 8192, None) == -5
    assert L.fpq_strerror(-2).decode().startswith("invalid ExMy")
    assert L.fpq_strerror(0) == b"ok"


def test_plan_query_and_format_range():
    L = B.lib()
    assert B.fpq_gemm_plan(8, 1280, 1280) == (B.FPQ_KERNEL_ROWS16, 1)
    assert B.fpq_gemm_plan(616, 320, 768) == (B.FPQ_KERNEL_SMALL_TILE, 1)
    assert B.fpq_gemm_plan(4096, 333, 640) == (B.FPQ_KERNEL_SMALL_TILE, 1)          # N not a multiple of 160
    k, s = B.fpq_gemm_plan(512, 1280, 5120)
    assert k == B.FPQ_KERNEL_128x160 and s > 1
    assert B.fpq_gemm_workspace_size(512, 1280, 5120, 0) == s * 512 * 1280 * 4
    k, s = B.fpq_conv2d_plan(8, 1280, 32, 32, 1280, 3, 3, 1, 1)
    assert k == B.FPQ_KERNEL_256x160 and s == 1
    p = B.fpq_plan_t()
    assert L.fpq_gemm_plan(0, 8, 8, C.byref(p)) == -4
    assert L.fpq_gemm_plan(8, 8, 8, None) == -1
    assert L.fpq_conv2d_plan(1, 16, 2, 2, 8, 3, 3, 1, 0, C.byref(p)) == -4
    # encodings whose largest value would overflow the encoder's fp32 rounding constant are rejected
    assert B.fpq_format_check((7, 0, 23, 0.0)) == 0 and B.fpq_format_check((7, 0, 22, 0.0)) == -2
    assert B.fpq_format_check((6, 1, -42, 0.0)) == 0 and B.fpq_format_check((6, 1, -43, 0.0)) == -2
    assert B.fpq_format_max(7, 0, 0) == 0.0
    assert B.fpq_format_check((5, 2, -64, 0.0)) == 0 and B.fpq_format_check((4, 3, -64, 0.0)) == 0


def test_launch_plan_query():
    """What runs, next to what the workspace is sized for: tiles over the wavefronts in place of slices where the grid is large enough, for
    stored and for added fp32 results in the exact mode, and nowhere else; the refusals of the layer calls."""
    E4M3, E2M1, E3M4, E3M0, E5M2 = synth.E4M3, synth.E2M1, synth.E3M4, synth.E3M0, synth.E5M2
    deep = (8, 1280, 16, 16, 1280, 3, 3, 1, 1)
    assert B.fpq_conv2d_plan(*deep) == (B.FPQ_KERNEL_128x160, 4)
    for fx, fw in ((E4M3, E4M3), (E4M3, E2M1), (E3M4, E3M0)):
        for add in (0, B.FPQ_OUT_ACCUMULATE):
            assert B.fpq_conv2d_launch_plan(*deep, fx, fw, B.FPQ_ACC_FP32 | add) == (B.FPQ_KERNEL_128x80, 1)
    assert B.fpq_conv2d_launch_plan(*deep, E4M3, E4M3, B.FPQ_ACC_FP8_MFMA) == B.fpq_conv2d_plan(*deep)
    assert B.fpq_conv2d_launch_plan(*deep, E5M2, E5M2) == (B.FPQ_KERNEL_128x160, 4)
    assert B.fpq_conv2d_launch_plan(1, 320, 64, 64, 320, 3, 3, 1, 1, E4M3, E4M3) == (B.FPQ_KERNEL_64x80, 1)
    few = (1, 2560, 8, 8, 1280, 3, 3, 1, 1)                           # slices stay where the tiles are few
    assert B.fpq_conv2d_launch_plan(*few, E4M3, E4M3) == B.fpq_conv2d_plan(*few) == (B.FPQ_KERNEL_128x160, 22)
    assert B.fpq_gemm_launch_plan(2048, 1280, 4096, E4M3, E2M1) == (B.FPQ_KERNEL_128x80, 1)
    assert B.fpq_gemm_launch_plan(128, 1280, 32768, E3M4, E3M4) == (B.FPQ_KERNEL_128x160, 32)
    # what other kernels serve
    assert B.fpq_gemm_launch_plan(8, 1280, 1280, E4M3, E4M3) == (B.FPQ_KERNEL_ROWS16, 1)
    assert B.fpq_gemm_launch_plan(8, 1280, 1280, E3M4, E3M0)[0] == B.FPQ_KERNEL_SMALL_TILE
    assert B.fpq_gemm_launch_plan(16384, 960, 320, E4M3, E4M3) == (B.FPQ_KERNEL_STRIP, 1)
    assert B.fpq_gemm_launch_plan(16384, 960, 320, E4M3, E4M3, B.FPQ_OUT_ACCUMULATE) == (B.FPQ_KERNEL_128x160, 1)
    assert B.fpq_conv2d_launch_plan(8, 64, 32, 32, 320, 7, 7, 1, 3, E4M3, E4M3) == (B.FPQ_KERNEL_SMALL_TILE, 1)   # 49 taps
    L, p, f = B.lib(), B.fpq_plan_t(), B.fmt(E4M3)
    assert L.fpq_gemm_launch_plan(8, 8, 16, f, f, 0, None) == -1
    assert L.fpq_gemm_launch_plan(0, 8, 16, f, f, 0, C.byref(p)) == -4
    assert L.fpq_gemm_launch_plan(8, 1 << 24, 16, f, f, 0, C.byref(p)) == -4
    assert L.fpq_gemm_launch_plan(8, 1 << 20, 4096, f, f, 0, C.byref(p)) == -4                 # 4 GiB of weights
    assert L.fpq_conv2d_launch_plan(1, 16, 2, 2, 8, 3, 3, 1, 0, f, f, 0, C.byref(p)) == -4
    assert L.fpq_gemm_launch_plan(8, 8, 16, B.fmt(E2M1), f, 0, C.byref(p)) == -8               # four-bit activations
    assert L.fpq_gemm_launch_plan(8, 8, 16, f, B.fmt((9, 1, 1, 0.0)), 0, C.byref(p)) == -2
    assert L.fpq_gemm_launch_plan(8, 8, 16, f, f, B.FPQ_ACT_SILU, C.byref(p)) == -8            # no stored result


def test_search_workspace_sizes():
    """The sizes the header states, in whole megabytes, and the least that is taken."""
    size = lambda n, e=4, j=111: B.fpq_search_workspace_size(n, e, j)
    assert [round(size(n) / 1e6) for n in (1572864, 8 * 320 * 64 * 64, 1 << 26, (1 << 26) + 1)] == [23, 47, 197, 42]
    assert size(2000) == 4352 + 4 * 444 + 16                   # one workgroup's sums, to whole 256 bytes


def test_plan_query_of_a_short_k():
    """Every output from one row of at most 320 codes: the kernel that keeps the weights in registers, from 144 pairs of 128 rows and
    64 columns on (NCHW results: from 32 channels on); with more than 64 and at most 128 codes, one step of the tiles, from 4 M values on."""
    strip = (B.FPQ_KERNEL_STRIP, 1)
    assert B.fpq_conv2d_plan(8, 320, 64, 64, 320, 1, 1, 1, 0) == strip
    assert B.fpq_gemm_plan(16384, 960, 320) == strip and B.fpq_gemm_plan(18432, 64, 16) == strip
    assert B.fpq_gemm_plan(17, 9216, 320) == strip and B.fpq_conv2d_plan(1, 3, 5, 5, 32, 1, 1, 1, 0) == strip
    assert B.fpq_gemm_plan(6250, 640, 128) == strip and B.fpq_gemm_plan(40000, 640, 128) == strip
    for plan in (B.fpq_gemm_plan(6249, 640, 128), B.fpq_gemm_plan(6249, 640, 80), B.fpq_gemm_plan(17, 9215, 320), B.fpq_gemm_plan(16384, 960, 336), B.fpq_gemm_plan(16, 9216, 320),
                 B.fpq_gemm_plan(18304, 64, 16), B.fpq_gemm_plan(18432, 63, 16), B.fpq_gemm_plan(16384, 1001, 320),
                 B.fpq_gemm_plan(1 << 20, 640, (1 << 32) + 320), B.fpq_conv2d_plan(1, 3, 5, 5, 31, 1, 1, 1, 0),
                 B.fpq_conv2d_plan(1, 3, 4, 4, 32, 1, 1, 1, 0), B.fpq_conv2d_plan(8, 16, 64, 64, 320, 3, 3, 1, 1),
                 B.fpq_conv2d_plan(8, 320, 64, 64, 320, 1, 1, 2, 0), B.fpq_conv2d_plan(8, 320, 64, 64, 320, 1, 1, 1, 1)):
        assert plan[0] != B.FPQ_KERNEL_STRIP


def test_workspace_holds_the_partial_sums_of_any_operands():
    """Formats of five exponent bits are not built on the small tiles: on widths of 160 they keep the 160-wide tiles and their
    slices, also where the hardware's formats take small tiles in fewer slices, or whole."""
    for M, N, K, slices in [(256, 1280, 11520, 11), (4096, 320, 2880, 2), (40, 1280, 5120, 5), (2048, 1280, 1280, 1),
                            (616, 320, 768, 1), (8, 1280, 11520, 1)]:
        most = max(slices, B.fpq_gemm_plan(M, N, K)[1])
        assert B.fpq_gemm_workspace_size(M, N, K, 0) == (most * M * N * 4 if most > 1 else 0), (M, N, K)


def test_noalloc_entry_validates_before_touching_the_gpu():
    L = B.lib()
    f = B.fmt(synth.E4M3)
    p = C.c_void_p(4096)
    assert L.fpq_gemm_noalloc(p, 1, f, 1.0, None, p, f, p, None, p, 1 << 20, 320, 4096, 0, None) == -6   # 4 GiB of codes
    assert L.fpq_gemm_noalloc(p, 0, f, 1.0, None, p, f, p, None, p, 0, 8, 32, 0, None) == 0
    assert L.fpq_gemm_noalloc(p, 0, f, 1.0, None, p, f, p, None, p, 8, 0, 32, 0, None) == -4
    assert L.fpq_strerror(-9).decode().startswith("packed weights")


def test_grouped_call_takes_the_problem_array_only():
    """The library reads device addresses from the array: other objects with a buffer are refused before that."""
    array = B.gemm_problems([])
    for other in (b"\0" * 72, bytearray(72), (C.c_int64 * 9)(), None, [1, 2], C.pointer((B.fpq_gemm_problem_t * 1)())):
        with pytest.raises(TypeError, match="gemm_problems"):
            B.fpq_gemm_grouped(other, 0, synth.E4M3, synth.E4M3)
    with pytest.raises(Exception) as e:                       # (what the CPU has instead of a stream, or no error on a GPU)
        B.fpq_gemm_grouped(array, 7, synth.E4M3, synth.E4M3)
        raise RuntimeError("taken")
    assert "gemm_problems" not in str(e.value)


def test_native_calls_that_do_not_load_name_the_cause(tmp_path):
    import shutil
    import subprocess
    import sys
    package = tmp_path / "paper_2408_06995_amd"
    package.mkdir()
    for f in ("__init__.py", "binding.py", "synth.py"):
        shutil.copy(os.path.join(ROOT, "paper_2408_06995_amd", f), package / f)
    ask = [sys.executable, "-c", "from paper_2408_06995_amd import binding as B\n"
           "try: B.fpq_gemm()\nexcept ImportError as e: print(e, '|', type(e.__cause__).__name__)"]
    run = lambda: subprocess.run(ask, cwd=tmp_path, capture_output=True, text=True, check=True).stdout
    assert "is not built" in run()
    (package / "_fpqcall.so").write_bytes(b"no library")
    out = run()
    assert "does not load" in out and "invalid ELF header" in out or "file too short" in out, out
