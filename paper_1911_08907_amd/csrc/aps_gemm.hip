// aps_gemm.hip -- low-precision GEMM: the C ABI entry point and the choice of
// the kernel.
#include "aps_gemm.hpp"

using namespace aps;

extern "C" int aps_lp_gemm(const float* A, int64_t lda, const float* B, int64_t ldb, float* C, int64_t ldc,
                           int32_t M, int32_t N, int32_t K, aps_format in_fmt, aps_format acc_fmt,
                           int32_t accumulator, void* stream) {
    if (M < 0 || N < 0 || K < 0 || M > APS_MAX_GEMM_DIM || N > APS_MAX_GEMM_DIM || K > APS_MAX_GEMM_DIM)
        return APS_ERR_SIZE;
    const bool has_out = (int64_t)M * N > 0;
    if (has_out && (!C || (K > 0 && (!A || !B)))) return APS_ERR_NULL;
    if (has_out && (ldc < N || (K > 0 && (lda < K || ldb < N)))) return APS_ERR_SIZE;
    int st = fmt_status(in_fmt);
    if (st != APS_OK) return st;
    st = fmt_status(acc_fmt);
    if (st != APS_OK) return st;
    if (accumulator != APS_ACC_SEQUENTIAL && accumulator != APS_ACC_KAHAN) return APS_ERR_UNSUPPORTED;
    // formats rounded in fp64 (class GEN) are not built into the GEMM
    if (make_fmtk(in_fmt).variant == V_GEN || make_fmtk(acc_fmt).variant == V_GEN) return APS_ERR_UNSUPPORTED;
    // the product of two input values must be exact in fp32, or round to zero anyway
    const int emin_in = 1 - in_fmt.bias, emin_acc = 1 - acc_fmt.bias;
    if (in_fmt.m > 11) return APS_ERR_UNSUPPORTED;
    if (2 * (emin_in - in_fmt.m) < -149 && 2 * (in_fmt.m + 1) > emin_acc - acc_fmt.m + 149) return APS_ERR_UNSUPPORTED;
    if (!has_out) return APS_OK;
    const FmtK fi = make_fmtk(in_fmt), fa = make_fmtk(acc_fmt);
    GemmArgs g{A, B, C, lda, ldb, ldc, M, N, K, 0, 0, 1.0f};
    // Pre-scale the staged operands by 2^ka and 2^kb (ka + kb = k) when both
    // stay below 2^128: a value below 2^(emax_in+1) times 2^(127-emax_in) does.
    const int room = 127 - fi.emax;
    int pm = GP_LDEXP;
    if (fa.k <= 2 * room) {
        g.ka = fa.k < room ? fa.k : room;
        g.kb = fa.k - g.ka;
        pm = GP_SCALED;
        // every product has at most 2(m_in+1) significant bits
        const int cls = fa.variant <= V_INT_M0 ? CLS_INT : (fa.variant <= V_TOP_M0 ? CLS_TOP : CLS_LOW);
        if (cls != CLS_INT && acc_fmt.m > 0 && 2 * (in_fmt.m + 1) <= acc_fmt.m + 1) pm = GP_FIT;
    }
    if (pm == GP_FIT) {
        // GP_GRID where the step's exponent Q is >= 0 (the format spans at
        // most 128 binades with its subnormals, so a staged product overflows
        // fp32 only where the format does) and the operands can carry
        // 2^(m - emin) between them as fp32 normals: staged values from the
        // input's smallest subnormal to below 2^128
        const int q = fa.emin + fa.k - acc_fmt.m;
        const int kq = acc_fmt.m - fa.emin;
        const int lo = -126 - (fi.emin - in_fmt.m), hi = 127 - fi.emax;
        const int ka = std::min(std::max(kq / 2, lo), hi), kb = kq - ka;
        if (q >= 0 && q <= 127 && kb >= lo && kb <= hi) {
            g.ka = ka;
            g.kb = kb;
            g.qs = pow2f_host(q);
            pm = GP_GRID;
        }
    }
    // GP_EXACT: each product fits the significand (pm is GP_FIT or GP_GRID, or
    // the class is INT) and is a multiple of the subnormal step
    if (pm != GP_LDEXP && acc_fmt.m > 0 && 2 * (in_fmt.m + 1) <= acc_fmt.m + 1 &&
        2 * (fi.emin - in_fmt.m) >= fa.emin - acc_fmt.m) {
        // products staged in the working domain (ka + kb = k, both >= 0, so
        // every staged value stays exact)
        g.ka = fa.k < room ? fa.k : room;
        g.kb = fa.k - g.ka;
        g.qs = 1.0f;
        // the largest product against the largest accumulator value, both exact in fp64
        const double top_in = std::ldexp(2.0 - std::ldexp(1.0, -in_fmt.m), fi.emax);
        const double top_acc = std::ldexp(2.0 - std::ldexp(1.0, -acc_fmt.m), fa.emax);
        pm = top_in * top_in <= top_acc ? GP_FMA : GP_EXACT;
    }
    if (acc_fmt.m == 7 && pm >= GP_GRID) pm = pm == GP_GRID ? GP_B7_GRID : (pm == GP_EXACT ? GP_B7_EXACT : GP_B7_FMA);
    if (pm == GP_FMA && acc_fmt.m > 10 && acc_fmt.m < 23) pm = GP_EXACT;  // adds in fp64: nothing to fuse
    if (pm == GP_FMA && acc_fmt.m == 23 && fa.variant != V_INT_EXACT) pm = GP_EXACT;
    const hipStream_t s = (hipStream_t)stream;
    const bool kahan = accumulator == APS_ACC_KAHAN;
    // the accumulator is IEEE half and every input value a half (at most 10
    // mantissa bits, at most 2^15 and no finer than half's step 2^-24); such
    // an input format is of class TOP or LOW
    const bool half_acc = acc_fmt.e == 5 && acc_fmt.m == 10 && acc_fmt.bias == 15;
    if (half_acc && in_fmt.m <= 10 && fi.emax <= 15 && fi.emin - in_fmt.m >= -24 && launch_gemm_half(kahan, s, g, fi))
        return launched();
    if (pm >= GP_B7_GRID)
        launch_gemm_b7(pm, kahan, s, g, fi, fa);
    else if (fa.variant <= V_INT_M0)
        launch_gemm_int(fa.variant, pm, kahan, s, g, fi, fa);
    else if (fa.variant <= V_TOP_M0)
        launch_gemm_top(fa.variant, pm, kahan, s, g, fi, fa);
    else
        launch_gemm_low(fa.variant, pm, kahan, s, g, fi, fa);
    return launched();
}
