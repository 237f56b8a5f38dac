// K-split-over-wavefronts kernel (gemm_wk_kernel.h), fp32 results.
#include "gemm_wk_kernel.h"

namespace fpq {

int launch_gemm_wk(const GemmArgs& a, hipStream_t st)
{
    if (a.acc_mode == FPQ_ACC_FP8_MFMA) {
        if (a.xkind == OPK_FP8 && a.wkind == OPK_FP8) return launch_wk_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA, false>(a, st);
        if (a.xkind == OPK_FP8 && a.wkind == OPK_FP4) return launch_wk_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA, false>(a, st);
        return FPQ_ERR_UNSUPPORTED;
    }
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP8) return launch_wk_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP32, false>(a, st);
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP4) return launch_wk_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP32, false>(a, st);
    if (a.xkind == OPK_HALF8 && a.wkind == OPK_HALF8) return launch_wk_shape<OPK_HALF8, OPK_HALF8, FPQ_ACC_FP32, false>(a, st);
    if (a.xkind == OPK_HALF8 && a.wkind == OPK_HALF4) return launch_wk_shape<OPK_HALF8, OPK_HALF4, FPQ_ACC_FP32, false>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
