// aps_gemm_low.hip -- low-precision GEMM: accumulators of class LOW.
#include "aps_gemm.hpp"

namespace aps {

void launch_gemm_low(int variant, int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                     const FmtK& fa) {
    if (variant == V_LOW_F32) launch_gemm_v<V_LOW_F32>(pm, kahan, s, g, fi, fa);
    if (variant == V_LOW_F64) launch_gemm_v<V_LOW_F64>(pm, kahan, s, g, fi, fa);
    if (variant == V_LOW_M0) launch_gemm_v<V_LOW_M0>(pm, kahan, s, g, fi, fa);
}

}  // namespace aps
