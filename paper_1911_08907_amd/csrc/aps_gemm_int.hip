// aps_gemm_int.hip -- low-precision GEMM: accumulators of e = 8, bias 127 (class INT).
#include "aps_gemm.hpp"

namespace aps {

void launch_gemm_int(int variant, int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                     const FmtK& fa) {
    if (variant == V_INT_F32) launch_gemm_v<V_INT_F32>(pm, kahan, s, g, fi, fa);
    if (variant == V_INT_F64) launch_gemm_v<V_INT_F64>(pm, kahan, s, g, fi, fa);
    if (variant == V_INT_EXACT) launch_gemm_v<V_INT_EXACT>(pm, kahan, s, g, fi, fa);
    if (variant == V_INT_M0) launch_gemm_v<V_INT_M0>(pm, kahan, s, g, fi, fa);
}

}  // namespace aps
