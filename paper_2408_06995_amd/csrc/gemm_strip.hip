// Weights-in-registers kernel for a short K: fp32 results, hardware encodings, and the choice of kernel.
#include "gemm_strip_kernel.h"

namespace fpq {

// Layers the kernel is built for (every output depends on one row of activations of at most 320 codes) and is the faster one for,
// against the 128 x 160, 128 x 64 and register-staged 64 x 64 tiles:
//   - codes out (feed-forward blocks of 64 to 20000 rows, K of 64 to 320: 1.13 to 2.2 times) and NCHW results of at least 32 channels
//     (1.2 to 2.3 times; 8 channels, an eighth of a strip: 0.9 to 1.0): all of them;
//   - results in rows: from 144 pairs of a strip and 128 rows on (1000 x 64 -> 2560 1.8, 16384 x 320 -> 960 1.3 times); below, layers
//     are at the launch floor, where the weights' way through LDS costs up to 1 us (500 x 256 -> 1000: 3.6 and 4.5 us).  Not strips
//     that are mostly empty, and not long rows that share lines at K above 256 (33000 x 320 -> 1001: 49.7 and 52.9 us).
bool gemm_strip_applicable(const GemmArgs& a)
{
    if (a.splits != 1 || a.accumulate || a.kh * a.kw != 1 || a.stride != 1 || a.pad != 0 || a.M <= 16 || a.Kreal > 320) return false;
    const bool native = a.xkind == OPK_FP8 && (a.wkind == OPK_FP8 || a.wkind == OPK_FP4);
    if (a.yq) return native && (a.ykind == 1 || a.act == 0);
    if (!native && (a.acc_mode == FPQ_ACC_FP8_MFMA || a.xkind != OPK_HALF8 || (a.wkind != OPK_HALF8 && a.wkind != OPK_HALF4))) return false;
    if (a.conv_out) return a.N >= 32;
    if (a.N < 64 || (a.N % 32 != 0 && a.N > 512 && a.Kreal > 256)) return false;
    return (int64_t)((a.M + 127) / 128) * ((a.N + 63) / 64) >= 144;
}

template <int XKIND, int WKIND, int ACC>
static int launch_strip_out(const GemmArgs& a, hipStream_t st)
{
    return a.conv_out ? launch_strip_k<XKIND, WKIND, ACC, STRIP_NCHW>(a, st) : launch_strip_k<XKIND, WKIND, ACC, STRIP_ROWS>(a, st);
}

int launch_gemm_strip(const GemmArgs& a, hipStream_t st)
{
    if (a.yq) return launch_gemm_strip_q(a, st);
    if (a.xkind == OPK_HALF8) return launch_gemm_strip_h(a, st);
    if (a.acc_mode == FPQ_ACC_FP8_MFMA)
        return a.wkind == OPK_FP8 ? launch_strip_out<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA>(a, st)
                                  : launch_strip_out<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA>(a, st);
    return a.wkind == OPK_FP8 ? launch_strip_out<OPK_FP8, OPK_FP8, FPQ_ACC_FP32>(a, st)
                              : launch_strip_out<OPK_FP8, OPK_FP4, FPQ_ACC_FP32>(a, st);
}

}  // namespace fpq
