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

template <int XKIND, int WKIND, int ACC>
static int launch_wk_group(const GroupedArgs& g, hipStream_t st)
{
    constexpr int smem = 4 * wk_wave_lds(2, kind_is_4bit(WKIND)) + 1024;
    int most = 0;
    for (int i = 0; i < g.count; ++i) {
        const int t = ((g.p[i].M + 63) / 64) * ((g.p[i].N + 63) / 64);
        most = t > most ? t : most;
    }
    auto kern = gemm_wk_grouped_kernel<2, XKIND, WKIND, ACC>;
    static std::atomic<uint64_t> allowed{0};
    if (!allow_dynamic_lds(reinterpret_cast<const void*>(kern), smem, allowed)) return FPQ_ERR_LAUNCH;
    hipLaunchKernelGGL(kern, dim3((unsigned)most, (unsigned)g.count), dim3(256), smem, st, g);
    return hipGetLastError() == hipSuccess ? FPQ_OK : FPQ_ERR_LAUNCH;
}

int launch_wk_grouped(const GroupedArgs& g, hipStream_t st)
{
    const GemmArgs& a = g.common;
    if (a.acc_mode == FPQ_ACC_FP8_MFMA)
        return a.wkind == OPK_FP8 ? launch_wk_group<OPK_FP8, OPK_FP8, FPQ_ACC_FP8_MFMA>(g, st)
                                  : launch_wk_group<OPK_FP8, OPK_FP4, FPQ_ACC_FP8_MFMA>(g, st);
    if (a.xkind == OPK_HALF8)
        return a.wkind == OPK_HALF8 ? launch_wk_group<OPK_HALF8, OPK_HALF8, FPQ_ACC_FP32>(g, st)
                                    : launch_wk_group<OPK_HALF8, OPK_HALF4, FPQ_ACC_FP32>(g, st);
    return a.wkind == OPK_FP8 ? launch_wk_group<OPK_FP8, OPK_FP8, FPQ_ACC_FP32>(g, st)
                              : launch_wk_group<OPK_FP8, OPK_FP4, FPQ_ACC_FP32>(g, st);
}

}  // namespace fpq
