// Weights-in-registers kernel for a short K: fp32 results, hardware encodings, and the choice of kernel.
#include "gemm_strip_kernel.h"
#include "strip_rule.h"

namespace fpq {

// Layers the kernel is built for (every output depends on one row of activations of at most 320 codes) and is the faster one for,
// against the 128 x 160, 128 x 64 and register-staged 64 x 64 tiles: codes out (416 layers of 17 to 60000 rows, K of 16 to 320: 1.26 to
// 1.37 times, none below 0.98) and NCHW results of at least 32 channels (104 layers: 1.46 times; 8 channels, an eighth of a strip:
// 0.9 to 1.0): all of them.  Results in rows: strip_rule.h.
bool gemm_strip_applicable(const GemmArgs& a)
{
    if (a.splits != 1 || a.accumulate || a.kh * a.kw != 1 || a.stride != 1 || a.pad != 0 || a.M <= 16 || a.Kreal > 320) return false;
    const bool native = a.xkind == OPK_FP8 && (a.wkind == OPK_FP8 || a.wkind == OPK_FP4);
    if (a.yq) return native && (a.ykind == 1 || a.act == 0);
    if (!native && (a.acc_mode == FPQ_ACC_FP8_MFMA || a.xkind != OPK_HALF8 || (a.wkind != OPK_HALF8 && a.wkind != OPK_HALF4))) return false;
    return a.conv_out ? a.N >= 32 : strip_rows(a.M, a.N, a.Kreal, native, a.wkind == OPK_FP4);
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
