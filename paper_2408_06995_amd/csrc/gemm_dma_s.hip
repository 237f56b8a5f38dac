// Large-tile kernel's pipeline on tiles for widths that are no multiple of 160 and for grids that the 160-wide tile would leave
// half empty, fp32 results: 128 x 64 (2 x 2 wavefronts of 64 x 32, three stages) and 128 x 128 (of 64 x 64, two stages), two
// workgroups per compute unit.  Any M and N: what a tile has beyond the matrix loads as zeros.  Bound by the conversion of codes ahead of the
// MFMAs.  Measured against the register-staged tiles that such shapes took before: 2048 x 1280 -> 1280 18.3 -> 13.6 us,
// 8 x 448 x 32 x 32 -> 448, 3 x 3: 54 -> 38 us, 12992 x 832 -> 576: 26 -> 18.5 us.
#include "gemm_dma_kernel.h"

namespace fpq {

template <int XKIND, int WKIND, int ACC>
static int launch_dma_s_shape(const GemmArgs& a, hipStream_t st)
{
    if (a.tile == TILE_128x64)
        return a.conv_out ? launch_dma_one<128, 64, 3, 2, XKIND, WKIND, ACC, true, false>(a, st)
                          : launch_dma_one<128, 64, 3, 2, XKIND, WKIND, ACC, false, false>(a, st);
    return a.conv_out ? launch_dma_one<128, 128, 2, 2, XKIND, WKIND, ACC, true, false>(a, st)
                      : launch_dma_one<128, 128, 2, 2, XKIND, WKIND, ACC, false, false>(a, st);
}

int launch_gemm_dma_s(const GemmArgs& a, hipStream_t st)
{
    if (a.acc_mode == FPQ_ACC_FP8_MFMA) {
        if (a.xkind == OPK_FP8 && a.wkind == OPK_FP8) return launch_dma_s_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA>(a, st);
        if (a.xkind == OPK_FP8 && a.wkind == OPK_FP4) return launch_dma_s_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA>(a, st);
        return FPQ_ERR_UNSUPPORTED;
    }
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP8) return launch_dma_s_shape<OPK_FP8, OPK_FP8, FPQ_ACC_FP32>(a, st);
    if (a.xkind == OPK_FP8 && a.wkind == OPK_FP4) return launch_dma_s_shape<OPK_FP8, OPK_FP4, FPQ_ACC_FP32>(a, st);
    if (a.xkind == OPK_HALF8 && a.wkind == OPK_HALF8) return launch_dma_s_shape<OPK_HALF8, OPK_HALF8, FPQ_ACC_FP32>(a, st);
    if (a.xkind == OPK_HALF8 && a.wkind == OPK_HALF4) return launch_dma_s_shape<OPK_HALF8, OPK_HALF4, FPQ_ACC_FP32>(a, st);
    return FPQ_ERR_UNSUPPORTED;
}

}  // namespace fpq
