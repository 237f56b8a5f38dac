// K-split-over-wavefronts kernel (gemm_wk_kernel.h), results that leave as codes for the next quantized layer.
#include "gemm_wk_kernel.h"

namespace fpq {

int launch_gemm_wk_q(const GemmArgs& a, hipStream_t st)
{
    if (a.xkind != OPK_FP8 || !a.yq) return FPQ_ERR_UNSUPPORTED;
    if (a.acc_mode == FPQ_ACC_FP8_MFMA) {
        if (a.wkind == OPK_FP8) return launch_wk_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA, true>(a, st);
        if (a.wkind == OPK_FP4) return launch_wk_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA, true>(a, st);
        return FPQ_ERR_UNSUPPORTED;
    }
    if (a.wkind == OPK_FP8) return launch_wk_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP32, true>(a, st);
    if (a.wkind == OPK_FP4) return launch_wk_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP32, true>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
