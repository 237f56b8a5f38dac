// Weights-in-registers kernel for a short K: operands moved into halves.
#include "gemm_strip_kernel.h"

namespace fpq {

template <int WKIND>
static int launch_strip_half(const GemmArgs& a, hipStream_t st)
{
    return a.conv_out ? launch_strip_k<OPK_HALF8, WKIND, FPQ_ACC_FP32, STRIP_NCHW>(a, st)
                      : launch_strip_k<OPK_HALF8, WKIND, FPQ_ACC_FP32, STRIP_ROWS>(a, st);
}

int launch_gemm_strip_h(const GemmArgs& a, hipStream_t st)
{
    return a.wkind == OPK_HALF4 ? launch_strip_half<OPK_HALF4>(a, st) : launch_strip_half<OPK_HALF8>(a, st);
}

}  // namespace fpq
