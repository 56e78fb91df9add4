// aps_gemm_half.hip -- low-precision GEMM: the IEEE half accumulator, on packed half arithmetic.
#include "aps_gemm.hpp"

namespace aps {

template <int VI, int HP, int TM, int TN, bool KAHAN>
static void launch_half_tile(hipStream_t s, const GemmArgs& g, const FmtK& fi) {
    hipLaunchKernelGGL((k_lp_gemm_h<KAHAN, VI, TM, TN, TM == 2 ? 32 : 16, HP>), gemm_grid(g, 16 * TM, 16 * TN),
                       dim3(BLOCK), 0, s, g, fi);
}

// The tiles (outputs per thread), measured on MI355X with 1-5-2 inputs, us
// (4x4 without the product test, which costs more than it saves in tiles so
// small that a wave seldom waits for the VALU; the others with it):
//                         8x8    8x4    4x4    2x2 | Kahan  8x4   4x4   2x2
//   4096 x 4096 x 1024    389    404    522    636         1096  1199  1247
//   2048 x 2048 x 512      81     71     79     92          161   164   170
//   1500 x 1300 x 800     120     87     74     80          158   139   139
//   1024 x 1024 x 1024    151    108     63     60          198   110   101
//   256 x 1000 x 2048     290    204    113     56          396   213    97
// The larger tile reads less of LDS and stages less per product, but needs
// three blocks (8 x 8: 152 VGPRs), or about two (8 x 4, 4 x 4), on every CU.
template <int VI, int HP>
static void launch_half(bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi) {
    constexpr int HP2 = HP == HP_TEST ? HP_ROUND : HP;
    const auto blocks = [&](int64_t gm, int64_t gn) { return gemm_padded(g, gm, gn) / (gm * gn); };
    // tiles that pad a narrow product by no more than a third over the smallest
    // (12 x 2^18 x 40 Kahan: 95 us at 8 x 4, whose rows are 128, 33 at 2 x 2)
    const auto fits = [&](int64_t gm, int64_t gn) { return 3 * gemm_padded(g, gm, gn) <= 4 * gemm_padded(g, 32, 32); };
    if (kahan) {
        if (blocks(128, 64) >= 512 && fits(128, 64))
            launch_half_tile<VI, HP, 8, 4, true>(s, g, fi);
        else
            launch_half_tile<VI, HP2, 2, 2, true>(s, g, fi);
    } else if (blocks(128, 128) >= 768 && fits(128, 128)) {
        launch_half_tile<VI, HP, 8, 8, false>(s, g, fi);
    } else if (blocks(128, 64) >= 448 && fits(128, 64)) {
        launch_half_tile<VI, HP, 8, 4, false>(s, g, fi);
    } else if (blocks(64, 64) >= 256 && fits(64, 64)) {
        launch_half_tile<VI, HP2, 4, 4, false>(s, g, fi);
    } else {
        launch_half_tile<VI, HP2, 2, 2, false>(s, g, fi);
    }
}

bool launch_gemm_half(bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi) {
#define APS_HK(VI, HP)                                \
    if (input_mode_is((VI), fi)) {                    \
        launch_half<(VI), (HP)>(kahan, s, g, fi);     \
        return true;                                  \
    }
    // 1-4-3: products have 8 significant bits, are multiples of 2^-18 and at most 240^2 < 65504
    APS_HK(VI_E5M2, HP_TEST) APS_HK(VI_E4M3, HP_FMA)
    APS_HK(V_TOP_F32, HP_ROUND) APS_HK(V_TOP_M0, HP_ROUND) APS_HK(V_LOW_F32, HP_ROUND) APS_HK(V_LOW_M0, HP_ROUND)
#undef APS_HK
    return false;
}

}  // namespace aps
