// aps_gemm_b7.hip -- low-precision GEMM: accumulators of 7 mantissa bits (bfloat16 among them).
#include "aps_gemm.hpp"

namespace aps {

void launch_gemm_b7(int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi, const FmtK& fa) {
    // V_INT_F32 stands for "m >= 1, no NaN flag": these modes use nothing else of the variant
#define APS_GB(PM, VI)                                                          \
    if (pm == (PM) && ((VI) < 0 || input_mode_is((VI), fi))) {                  \
        launch_gemm<V_INT_F32, (PM), (VI)>(kahan, s, g, fi, fa);          \
        return;                                                                 \
    }
    APS_GB(GP_B7_FMA, VI_E5M2) APS_GB(GP_B7_FMA, VI_E4M3) APS_GB(GP_B7_FMA, V_TOP_F32) APS_GB(GP_B7_FMA, V_LOW_F32)
    APS_GB(GP_B7_FMA, -1)
    APS_GB(GP_B7_GRID, VI_E5M2) APS_GB(GP_B7_GRID, VI_E4M3) APS_GB(GP_B7_GRID, -1)
    APS_GB(GP_B7_EXACT, -1)
#undef APS_GB
}

}  // namespace aps
