// Small tiles of the large-tile kernel's pipeline (see gemm_dma_s.hip), results that leave as codes.
#include "gemm_dma_kernel.h"

namespace fpq {

template <int XKIND, int WKIND, int ACC>
static int launch_dma_sq_shape(const GemmArgs& a, hipStream_t st)
{
    if (a.tile == TILE_128x64)
        return a.conv_out ? launch_dma_one<128, 64, 3, 2, XKIND, WKIND, ACC, true, true>(a, st)
                          : launch_dma_one<128, 64, 3, 2, XKIND, WKIND, ACC, false, true>(a, st);
    return a.conv_out ? launch_dma_one<128, 128, 2, 2, XKIND, WKIND, ACC, true, true>(a, st)
                      : launch_dma_one<128, 128, 2, 2, XKIND, WKIND, ACC, false, true>(a, st);
}

int launch_gemm_dma_sq(const GemmArgs& a, hipStream_t st)
{
    if (a.xkind != OPK_FP8 || !a.yq) return FPQ_ERR_UNSUPPORTED;
    if (a.acc_mode == FPQ_ACC_FP8_MFMA) {
        if (a.wkind == OPK_FP8) return launch_dma_sq_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA>(a, st);
        if (a.wkind == OPK_FP4) return launch_dma_sq_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA>(a, st);
        return FPQ_ERR_UNSUPPORTED;
    }
    if (a.wkind == OPK_FP8) return launch_dma_sq_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP32>(a, st);
    if (a.wkind == OPK_FP4) return launch_dma_sq_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP32>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
