// The kernel of gemm_wk16_kernel.h, operands with a hardware conversion.
#include "gemm_wk16_kernel.h"

namespace fpq {

int launch_gemm_wk16(const GemmArgs& a, hipStream_t st)
{
    if (a.xkind == OPK_HALF8) return launch_gemm_wk16_h(a, st);
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP8) return launch_wk16_shape<OPK_FP8, OPK_FP8>(a, st);
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP4) return launch_wk16_shape<OPK_FP8, OPK_FP4>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
