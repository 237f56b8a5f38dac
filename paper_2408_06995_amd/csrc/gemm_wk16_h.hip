// The kernel of gemm_wk16_kernel.h, operands moved into halves.
#include "gemm_wk16_kernel.h"

namespace fpq {

int launch_gemm_wk16_h(const GemmArgs& a, hipStream_t st)
{
    if (a.wkind == OPK_HALF8) return launch_wk16_shape<OPK_HALF8, OPK_HALF8>(a, st);
    if (a.wkind == OPK_HALF4) return launch_wk16_shape<OPK_HALF8, OPK_HALF4>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
