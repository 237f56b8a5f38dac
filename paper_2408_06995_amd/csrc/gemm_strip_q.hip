// Weights-in-registers kernel for a short K: results that leave as codes.
#include "gemm_strip_kernel.h"

namespace fpq {

int launch_gemm_strip_q(const GemmArgs& a, hipStream_t st)
{
    if (a.acc_mode == FPQ_ACC_FP8_MFMA)
        return a.wkind == OPK_FP8 ? launch_strip_k<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA, STRIP_CODES>(a, st)
                                  : launch_strip_k<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA, STRIP_CODES>(a, st);
    return a.wkind == OPK_FP8 ? launch_strip_k<OPK_FP8, OPK_FP8, FPQ_ACC_FP32, STRIP_CODES>(a, st)
                              : launch_strip_k<OPK_FP8, OPK_FP4, FPQ_ACC_FP32, STRIP_CODES>(a, st);
}

}  // namespace fpq
