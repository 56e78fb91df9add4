// aps_gemm.hpp -- the kernels of the GEMM on a multiply-accumulate unit of a
// chosen low precision, CPD's low-precision-accumulator GEMM (Sec. 5), and
// the launchers that the instance files (aps_gemm_*.hip) define.
#pragma once

#include <type_traits>

#include "aps_common.hpp"

namespace aps {

// ================================================== K6: low-precision GEMM

struct GemmArgs {
    const float* __restrict__ A;
    const float* __restrict__ B;
    float* __restrict__ C;
    int64_t lda, ldb, ldc;
    int32_t M, N, K;
    int32_t ka, kb;  // staged A and B carry 2^ka, 2^kb (ka + kb = k of the accumulator, or both 0)
    float qs;        // grid modes: 2^Q, the accumulator's subnormal step in its working domain
};

// How a product reaches the accumulator's working domain and is rounded, and
// for the last three how each add is rounded.
enum GemmProduct {
    GP_LDEXP = 0,    // operands native: fl32(a * b) then 2^k, rounded (quant)
    GP_SCALED = 1,   // operands pre-scaled at staging: a_w * b_w rounded (quant_w)
    GP_FIT = 2,      // pre-scaled, and every product fits the significand (quant_fit)
    GP_GRID = 3,     // as GP_FIT, staged so that the subnormal step is 1: rint, then 2^Q
    GP_EXACT = 4,    // pre-scaled, every product is a format value or overflows: no rounding
    GP_FMA = 5,      // GP_EXACT, and no product overflows: multiply and add in one fma
    GP_B7_GRID = 6,  // GP_GRID, GP_EXACT and GP_FMA into an accumulator of 7 mantissa
    GP_B7_EXACT = 7, // bits: each add rounded by the hardware's conversion to bfloat16
    GP_B7_FMA = 8,
};

// Seven mantissa bits.  In the working domain the format's overflow sits at
// fp32's, and a sum of two format values is either below 2^emin, where it is
// an exact multiple of the subnormal step and has at most 7 significant
// bits, or rounds to 8 significant bits, ties to even: at every magnitude
// what fp32's conversion to bfloat16 does (subnormals and overflow to INF
// included; the accumulator 1-8-7 is bfloat16 itself).  The fp32 add of two
// such values rounded once more is the rounded exact sum (24 >= 2 * 8 + 2).
// The conversion of {0, x} leaves R(x) in the register's high half over a
// zero low half, which is R(x) as fp32: one instruction per add.  Taking two
// adds per conversion and unpacking them costs the same issue cycles (the
// conversion issues at half the rate of the shift and the mask) in one more
// instruction per add.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float round_b7(float x) {
    return __builtin_bit_cast(float, __builtin_convertvector(f32x2{0.0f, x}, bf16x2));
}

// GP_EXACT.  When every product of two input values fits the accumulator's
// significand and is a multiple of its subnormal step (the square of the
// input's smallest subnormal is), every product is already a format value,
// or beyond the largest one, where the working domain makes it INF as fp32
// does: the exact fp32 product is its own rounding.  When the square of the
// input's largest value is a format value too, none overflows, and fl32(s +
// a * b) with the product unrounded is one fma (GP_FMA).

// GP_GRID.  A product of two input values that fits the accumulator's
// significand is, from 2^emin up, already a multiple of the accumulator's
// subnormal step 2^(emin - m); below 2^emin the format rounds it to the
// nearest such multiple, ties to even.  So on a scale where that step is 1
// its rounding is one round-to-nearest-even to an integer at every
// magnitude, with no compare and select between the normal and subnormal
// cases.  The operands are staged with 2^(m - emin) between them, the
// product is rounded by rint, and 2^Q (Q = the step's exponent in the
// working domain, >= 0) carries it into the working domain: exactly, or to
// INF where the product overflows the format, as the format's own
// overflow threshold sits at fp32's there.  A staged product below 2^-126
// is below 1/2 and rounds to a signed zero whatever fp32 made of it.

// Input format 1-5-2 with bias 15 has the bit layout and value set of the
// OCP E5M2 8-bit float.  The hardware's conversion of fp32 to it (round to
// nearest even, no saturation: beyond the largest finite value the result is
// INF, a NaN stays NaN, subnormals kept) and back to fp32 is this format's
// cast exactly (round2_e5m2); the two agree on every fp32 bit pattern.
constexpr int VI_E5M2 = 100;

// Input format 1-4-3 with bias 7 shares its layout, subnormals and rounding
// with the OCP E4M3 8-bit float below 248; E4M3 has no INF and goes on to
// 448, so from 248 up (the tie at 248 rounds to 256) the cast is INF with the
// input's sign, which also covers an INF input.  With that one select the
// round trip is this format's cast on every fp32 bit pattern.
constexpr int VI_E4M3 = 101;

__device__ __forceinline__ void cast_e4m3x2(float x0, float x1, float& r0, float& r1) {
    const int pk = __builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false);  // bytes 0 and 1
    const f32x2 v = __builtin_amdgcn_cvt_pk_f32_fp8(pk, false);
    r0 = __builtin_fabsf(x0) >= 248.0f ? __builtin_copysignf(__builtin_inff(), x0) : v[0];
    r1 = __builtin_fabsf(x1) >= 248.0f ? __builtin_copysignf(__builtin_inff(), x1) : v[1];
}

// The launch's input mode: a hardware conversion, or the format's class.
inline bool input_mode_is(int vi, const FmtK& f) {
    if (vi == VI_E5M2) return f.hw == HW_E5M2;
    if (vi == VI_E4M3) return f.hw == HW_E4M3;
    return f.variant == vi;
}

// Four input values cast to the input format (native values): by a hardware
// conversion (E5M2, E4M3), straight to the class VI when the launch knows
// it, or through the switch over classes.
template <int VI>
__device__ __forceinline__ f4 cast_in4(const f4& x, const FmtK& fi) {
    if constexpr (VI == VI_E5M2 || VI == VI_E4M3) {
        float r0, r1, r2, r3;
        if constexpr (VI == VI_E5M2) {
            round2_e5m2(x.x, x.y, r0, r1);
            round2_e5m2(x.z, x.w, r2, r3);
        } else {
            cast_e4m3x2(x.x, x.y, r0, r1);
            cast_e4m3x2(x.z, x.w, r2, r3);
        }
        return f4{r0, r1, r2, r3};
    } else if constexpr (VI < 0) {
        return f4{quant_any(x.x, fi.k, fi), quant_any(x.y, fi.k, fi), quant_any(x.z, fi.k, fi),
                  quant_any(x.w, fi.k, fi)};
    } else {
        return f4{quant_native<VI>(x.x, fi.k, fi), quant_native<VI>(x.y, fi.k, fi), quant_native<VI>(x.z, fi.k, fi),
                  quant_native<VI>(x.w, fi.k, fi)};
    }
}

// Four values times 2^k, exact: the hardware modes' k lies in fp32's normal
// range, where a multiply issues at twice the rate of an ldexp.
template <int VI>
__device__ __forceinline__ f4 scale4(const f4& v, int k) {
    if constexpr (VI == VI_E5M2 || VI == VI_E4M3) {
        return v * u2f((uint32_t)(k + 127) << 23);
    } else {
        return f4{__builtin_amdgcn_ldexpf(v.x, k), __builtin_amdgcn_ldexpf(v.y, k), __builtin_amdgcn_ldexpf(v.z, k),
                  __builtin_amdgcn_ldexpf(v.w, k)};
    }
}

// The fp32 sum of two accumulator values rounded to the format (the classes
// whose adds need no fp64, m >= 1).
template <int V>
__device__ __forceinline__ float round_sum(float x, const FmtK& f) {
    if constexpr (VT<V>::acc == ACC_EXACT) {
        return x;
    } else {
        const uint32_t b = f2u(x);
        return u2f((b + f.half + __builtin_amdgcn_ubfe(b, f.sh, 1u)) & f.mask);
    }
}

// 16 bytes at any 4-byte alignment: rows of A, B and C start anywhere.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// Makes v's value needed here, without an instruction.
template <class T>
__device__ __forceinline__ void pin(T& v) {
    asm volatile("" : "+v"(v));
}

// The shape of a block's work: TM x TN outputs per thread, 16 x 16 threads,
// k-tiles of GK.
template <int TM, int TN, int GK_>
struct GemmTile {
    static constexpr int GM = 16 * TM, GN = 16 * TN;  // output tile GM x GN per block
    static constexpr int GK = GK_;
    static constexpr int FA = TM * GK / 64;  // 16-byte loads of A per thread and k-tile
    static constexpr int FB = TN * GK / 64;  // and of B
    static constexpr int TPA = GK / 4;       // threads that stage FA neighbouring rows of A, four k each
    static constexpr int TPB = GN / 4;       // threads that stage one row of B, four columns each
    static constexpr int RB = BLOCK / TPB;   // rows of B between a thread's loads
};

// A thread's loads of A and B, one k-tile at a time.  Every k-tile that ends
// three or more k before the last is read by unconditional 16-byte loads:
// rows of A past the last one read the last, and columns of B past the last
// one whatever follows in the matrix (such outputs are not stored), by offsets
// held to B's last four elements.  No column of B is held back so: in its
// first K-3 rows the four from column b (a multiple of 4 below N) start no
// later than (K-4) ldb + b <= (K-1) ldb + N-4, since b+4-N <= 3 <= 3 ldb.  One
// row more would not do for N = 1 and ldb < 3.  The last k-tile, and the one
// before it where the last holds one or two k, are read element by element
// with the indices clamped.
template <class D>
struct GemmLoads {
    const float* pa[D::FA];
    int64_t ob, last;  // offset of the first of B's four columns, and of the last four elements of B
    f4 ra[D::FA], rb[D::FB];

    __device__ __forceinline__ void init(const GemmArgs& g, int64_t m0, int64_t n0) {
        const int t = threadIdx.x;
#pragma unroll
        for (int r = 0; r < D::FA; ++r)
            pa[r] = g.A + min(m0 + t / D::TPA * D::FA + r, (int64_t)g.M - 1) * g.lda + t % D::TPA * 4;
        ob = (int64_t)(t / D::TPB) * g.ldb + n0 + t % D::TPB * 4;
        last = (int64_t)(g.K - 1) * g.ldb + g.N - 4;
    }
    // the k-tile from k0 on; tiles are fetched in order
    __device__ __forceinline__ void fetch(const GemmArgs& g, int k0, int64_t n0) {
        if (k0 + D::GK + 2 < g.K) {
#pragma unroll
            for (int r = 0; r < D::FA; ++r) {
                ra[r] = *(const f4u*)pa[r];
                pa[r] += D::GK;
            }
#pragma unroll
            for (int r = 0; r < D::FB; ++r) rb[r] = *(const f4u*)(g.B + min(ob + r * D::RB * g.ldb, last));
            ob += D::GK * g.ldb;
            return;
        }
        int t = threadIdx.x;
        pin(t);  // keeps this path's addresses out of the registers of the k loop
        const int k = k0 + t % D::TPA * 4;
#pragma unroll
        for (int r = 0; r < D::FA; ++r) {
#pragma unroll
            for (int q = 0; q < 4; ++q) ra[r][q] = pa[r][min(k + q, g.K - 1) - k];
            pa[r] += D::GK;
        }
#pragma unroll
        for (int r = 0; r < D::FB; ++r) {
            const float* row = g.B + min(k0 + t / D::TPB + r * D::RB, g.K - 1) * g.ldb;
#pragma unroll
            for (int q = 0; q < 4; ++q) rb[r][q] = row[min((int)n0 + t % D::TPB * 4 + q, g.N - 1)];
        }
    }
};

template <int N>
struct FVec {
    using T = float __attribute__((ext_vector_type(N)));
};

// One block computes a GM x GN tile of C.  Each k-tile of A and B is cast to
// the input format while it is staged into LDS (A transposed, so a thread's
// TM rows are read together); each thread then runs TM * TN independent chains,
// one per output, adding its products in k order.  The next k-tile's loads
// are issued before this tile's math and cast after it, into the other of
// two LDS buffers, so a wave never waits for memory in between and a k-tile
// costs one barrier.  Rows and columns past C are computed from the last one
// and not stored.
template <int V, bool KAHAN, int PM, int VI, int TM, int TN, int GK>
__global__ __launch_bounds__(BLOCK) void k_lp_gemm(GemmArgs g, FmtK fi, FmtK fa) {
    using D = GemmTile<TM, TN, GK>;
    using tm = typename FVec<TM>::T;
    using tn = typename FVec<TN>::T;
    // LDS row strides: A's spreads the transposed staging writes over the banks,
    // both keep the vector reads aligned
    constexpr int LA = D::GM + (TM < 4 ? TM : 4), LB = D::GN + 4;
    constexpr bool B7 = PM >= GP_B7_GRID;
    constexpr bool FMA = PM == GP_FMA || PM == GP_B7_FMA;
    __shared__ __align__(16) float As[2][GK][LA];  // As[.][k][m]
    __shared__ __align__(16) float Bs[2][GK][LB];  // Bs[.][k][n]
    const int t = threadIdx.x;
    const int tx = t & 15, ty = t >> 4;
    const int sam = t / D::TPA * D::FA, sak = t % D::TPA * 4;  // staged A: rows sam.., k sak..sak+3
    const int sbk = t / D::TPB, sbn = t % D::TPB * 4;          // staged B: rows sbk.., columns sbn..sbn+3
    // x: column of tiles, y: row of tiles (a grid's y extent is limited to 65535
    // blocks: a block takes further rows of tiles where there are more)
    const int64_t n0 = (int64_t)blockIdx.x * D::GN;
    for (int64_t m0 = (int64_t)blockIdx.y * D::GM; m0 < g.M; m0 += (int64_t)gridDim.y * D::GM) {
        float s[TM][TN], c[TM][TN];
        uint64_t bad[TM][TN];  // m = 0: the lanes of the wave whose chain met a NaN
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                s[i][j] = 0.0f;
                c[i][j] = 0.0f;
                bad[i][j] = 0;
            }
        GemmLoads<D> ld;
        auto put = [&](int buf) {
            f4 a[D::FA];
#pragma unroll
            for (int r = 0; r < D::FA; ++r) a[r] = scale4<VI>(cast_in4<VI>(ld.ra[r], fi), g.ka);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                typename FVec<D::FA>::T v;
#pragma unroll
                for (int r = 0; r < D::FA; ++r) v[r] = a[r][q];
                *(typename FVec<D::FA>::T*)&As[buf][sak + q][sam] = v;
            }
#pragma unroll
            for (int r = 0; r < D::FB; ++r)
                *(f4*)&Bs[buf][sbk + r * D::RB][sbn] = scale4<VI>(cast_in4<VI>(ld.rb[r], fi), g.kb);
        };
        // one k: the products of a thread's TM rows and TN columns join their chains
        auto mac = [&](const tm& a, const tn& b, bool first) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    // exact fp32 product of two input-format values, cast to the accumulator
                    float p = 0.0f;
                    bool nan = false;
                    if constexpr (PM == GP_LDEXP)
                        p = quant<V>(a[i] * b[j], fa.k, fa, nan);
                    else if constexpr (PM == GP_SCALED)
                        p = quant_w<V>(a[i] * b[j], fa, nan);
                    else if constexpr (PM == GP_FIT)
                        p = quant_fit<V>(a[i] * b[j], fa);
                    else if constexpr (PM == GP_GRID || PM == GP_B7_GRID)
                        p = __builtin_rintf(a[i] * b[j]) * g.qs;
                    else if constexpr (!FMA)
                        p = a[i] * b[j];
                    if (first) {  // an output's chain starts with its first product
                        s[i][j] = FMA ? a[i] * b[j] : p;
                    } else if constexpr (B7 || FMA) {
                        // R(s + x), or Kahan's step with every operation rounded
                        auto rnd = [&](float x) { return B7 ? round_b7(x) : round_sum<V>(x, fa); };
                        if constexpr (KAHAN) {
                            const float y = rnd(FMA ? __builtin_fmaf(a[i], b[j], -c[i][j]) : p - c[i][j]);
                            const float u = rnd(s[i][j] + y);
                            c[i][j] = rnd(rnd(u - s[i][j]) - y);
                            s[i][j] = u;
                        } else {
                            s[i][j] = rnd(FMA ? __builtin_fmaf(a[i], b[j], s[i][j]) : s[i][j] + p);
                        }
                    } else {
                        chain_step<V, KAHAN>(s[i][j], c[i][j], p, fa, nan);
                    }
                    if constexpr (VT<V>::m0) {
                        // a wave's mask in scalar registers, due here: a flag per lane the
                        // compiler tests after the unrolled steps, with every product and sum
                        // of theirs held in registers
                        bad[i][j] |= __ballot(nan);
                        asm volatile("" : "+s"(bad[i][j]));
                    }
                }
        };
        // NK steps of the staged k-tile from its row kr on; software-pipelined:
        // step kk+1's LDS reads are issued before step kk's math
        auto steps = [&](auto nk, int buf, int kr, bool first) {
            constexpr int NK = decltype(nk)::value;
            tm av = *(const tm*)&As[buf][kr][ty * TM];
            tn bv = *(const tn*)&Bs[buf][kr][tx * TN];
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                tm an = av;
                tn bn = bv;
                if (kk + 1 < NK) {
                    an = *(const tm*)&As[buf][kr + kk + 1][ty * TM];
                    bn = *(const tn*)&Bs[buf][kr + kk + 1][tx * TN];
                }
                __builtin_amdgcn_sched_barrier(0);
                mac(av, bv, kk == 0 && first);
                av = an;
                bv = bn;
            }
        };
        if (g.K > 0) {
            ld.init(g, m0, n0);
            ld.fetch(g, 0, n0);
            put(0);
        }
        __syncthreads();
        int buf = 0;
        int k0 = 0;
        for (; k0 + GK <= g.K; k0 += GK, buf ^= 1) {
            const bool more = k0 + GK < g.K;
            if (more) ld.fetch(g, k0 + GK, n0);  // in flight during this tile's math
            steps(std::integral_constant<int, GK>{}, buf, 0, k0 == 0);
            // the chains end here: without this the compiler sinks the math below the
            // staging, with every LDS read's value held in registers
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    pin(s[i][j]);
                    if constexpr (KAHAN) pin(c[i][j]);
                }
            if (more) put(buf ^ 1);
            __syncthreads();
        }
        // the rest of K, fewer than GK steps
        int kr = 0;
#pragma unroll 1
        for (; k0 + kr + 8 <= g.K; kr += 8) steps(std::integral_constant<int, 8>{}, buf, kr, k0 + kr == 0);
#pragma unroll 1
        for (; k0 + kr < g.K; ++kr) steps(std::integral_constant<int, 1>{}, buf, kr, k0 + kr == 0);
        __syncthreads();  // before another tile is staged
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t m = m0 + ty * TM + i;
            if (m >= g.M) continue;
            float* crow = g.C + m * g.ldc;
            float o[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j)
                o[j] = __builtin_amdgcn_ldexpf(finish<V>(s[i][j], (bad[i][j] >> (t & 63)) & 1u), -fa.k);
            const int64_t n = n0 + tx * TN;
            if (TN >= 4 && n + TN <= g.N) {
#pragma unroll
                for (int j = 0; j + 3 < TN; j += 4) *(f4u*)(crow + n + j) = f4{o[j], o[j + 1], o[j + 2], o[j + 3]};
            } else {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (n + j < g.N) crow[n + j] = o[j];
            }
        }
    }
}

// ===================================== K6h: the accumulator is IEEE half
//
// When the accumulator is the half-precision format (e = 5, m = 10, bias
// 15) and every input value is a half, the hardware's half-precision
// multiply and add are the emulated unit: each rounds its exact result to
// nearest even, with subnormals and overflow to INF, as the format does.
// So the products and the chain run in packed halves, one multiply and one
// add (Kahan: one multiply, four adds) per two outputs, with no bit
// manipulation.  A multiply and the add that follows it may fuse only where
// the product is a half: then R(s + a * b) = R(s + R(a * b)).
enum HalfProduct {
    HP_ROUND = 0,  // multiply, then add
    HP_FMA = 1,    // every product of two input values is a half: one fma
    HP_TEST = 2,   // tested per k-step: one fma where all of a wave's products are halves
};

template <int N>
struct HVec {
    using T = _Float16 __attribute__((ext_vector_type(N)));
};

// The 1-5-2 codes of four values, one per byte (E5M2's bits).
__device__ __forceinline__ uint32_t codes_e5m2(const f4& x) {
    const int lo = __builtin_amdgcn_cvt_pk_bf8_f32(x.x, x.y, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(x.z, x.w, lo, true);
}

// |v| * 2^16 of a code's value v as an integer, OR-ed into o: for a finite
// 1-5-2 value (a multiple of 2^-16 below 2^16) its fixed-point form, so that
// the OR over a group holds the group's lowest and highest set bit.  The
// conversion saturates, so INF counts as all bits, and takes NaN to 0 (with a
// NaN operand both forms of the multiply-accumulate are NaN).
__device__ __forceinline__ uint32_t fixed_bits(float v) {
    uint32_t r;
    asm("v_cvt_u32_f32 %0, |%1|" : "=v"(r) : "v"(v));
    return r;
}

__device__ __forceinline__ void or_fixed16(uint32_t codes, uint32_t o[4]) {
    const f32x2 lo = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(codes, 65536.0f, false);
    const f32x2 hi = __builtin_amdgcn_cvt_scalef32_pk_f32_bf8(codes, 65536.0f, true);
    o[0] |= fixed_bits(lo[0]);
    o[1] |= fixed_bits(lo[1]);
    o[2] |= fixed_bits(hi[0]);
    o[3] |= fixed_bits(hi[1]);
}

// v OR-ed over the lanes of a 16-lane row that differ in the bits of STEPS
// (rotations within the row by 8, 4, 2, 1).
template <int STEPS>
__device__ __forceinline__ uint32_t row_or(uint32_t v) {
    if constexpr (STEPS & 8) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xF, 0xF, true);
    if constexpr (STEPS & 4) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xF, 0xF, true);
    if constexpr (STEPS & 2) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xF, 0xF, true);
    if constexpr (STEPS & 1) v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, true);
    return v;
}

// One block computes a GM x GN tile of C, as k_lp_gemm does: two LDS buffers,
// the next k-tile in flight during this one's math.  A thread stages FA
// neighbouring rows of A, so its writes into the transposed tile are FA
// halves wide.
//
// HP_TEST (1-5-2 inputs).  A product of two of its values is a half unless
// it has a bit below 2^-24 or reaches 2^16.  While a k-tile is staged, the
// fixed-point forms of the values are OR-ed per k over the rows of each
// wave's part of the tile and over the tile's columns; the lowest and highest
// set bits of the two words bound every product of that k in the wave.  With
// activations ~ N(0, 1) and weights ~ N(0, 0.02^2) 88 % of the k-steps pass
// and take one packed fma per two outputs; the others multiply, then add.
// The test costs about a tenth of a k-tile's math: while fewer than a quarter
// of a tile's steps pass, only every eighth tile is tested (products that
// all lie below 2^-24: 2048 x 2048 x 512 in 96 us, 105 with every tile tested).
template <bool KAHAN, int VI, int TM, int TN, int GK, int HP>
__global__ __launch_bounds__(BLOCK) void k_lp_gemm_h(GemmArgs g, FmtK fi) {
#pragma clang fp contract(off)
    using D = GemmTile<TM, TN, GK>;
    using hm = typename HVec<TM>::T;
    using hn = typename HVec<TN>::T;
    using hf = typename HVec<D::FA>::T;
    constexpr int FA = D::FA, FB = D::FB;
    constexpr int LA = D::GM + 8, LB = D::GN + 8;  // LDS row strides: spread the staging writes over the banks
    static_assert(HP != HP_TEST || GK == 16, "a k-tile's test is one 16-lane row");
    __shared__ __align__(16) _Float16 As[2][GK][LA];  // As[.][k][m]
    __shared__ __align__(16) _Float16 Bs[2][GK][LB];  // Bs[.][k][n]
    __shared__ __align__(16) uint32_t orA[2][HP == HP_TEST ? 4 : 1][4][GK];  // [.][wave][16-lane row][k]
    __shared__ uint32_t orB[2][HP == HP_TEST ? GK : 1][2];                   // [.][k][half of the columns]
    __shared__ uint32_t passed[2];  // k-steps of wave 0 that passed in the last tested k-tile
    const int t = threadIdx.x;
    const int tx = t & 15, ty = t >> 4;
    const int sam = t / D::TPA * FA, sak = t % D::TPA * 4;  // staged A: rows sam..sam+FA-1, k sak..sak+3
    const int sbk = t / D::TPB, sbn = t % D::TPB * 4;       // staged B: rows sbk.., columns sbn..sbn+3
    const int64_t n0 = (int64_t)blockIdx.x * D::GN;
    for (int64_t m0 = (int64_t)blockIdx.y * D::GM; m0 < g.M; m0 += (int64_t)gridDim.y * D::GM) {
        // output (ty*TM + i, tx*TN + 2*h + e) is element e of s[i][h]
        h2 s[TM][TN / 2], c[KAHAN ? TM : 1][TN / 2];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int h = 0; h < TN / 2; ++h) {
                s[i][h] = g.K > 0 ? h2{-0.0f16, -0.0f16} : h2{0, 0};
                if constexpr (KAHAN) c[i][h] = h2{0, 0};
            }
        // the chain starts with its first product and no compensation: from s = -0
        // the first step gives s = p (signs of zero included), and c is cleared after it
        auto clear_c = [&]() {
            if constexpr (KAHAN)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h) c[i][h] = h2{0, 0};
        };
        GemmLoads<D> ld;
        auto put = [&](int buf, bool test) {
            if constexpr (VI == VI_E5M2) {
                // 1-5-2 codes are the top bytes of the same values as halves
                uint32_t ca[FA], cb[FB];
#pragma unroll
                for (int r = 0; r < FA; ++r) ca[r] = codes_e5m2(ld.ra[r]);
#pragma unroll
                for (int r = 0; r < FB; ++r) cb[r] = codes_e5m2(ld.rb[r]);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if constexpr (FA == 2)  // {0, code q of row 0, 0, code q of row 1}
                        *(uint32_t*)&As[buf][sak + q][sam] =
                            __builtin_amdgcn_perm(ca[1], ca[0], 0x040C000Cu + 0x01000100u * q);
                    else
                        *(uint16_t*)&As[buf][sak + q][sam] = (uint16_t)__builtin_amdgcn_perm(0, ca[0], 0x0C0C000Cu + 0x100u * q);
                }
#pragma unroll
                for (int r = 0; r < FB; ++r)
                    *(u2v*)&Bs[buf][sbk + r * D::RB][sbn] =
                        u2v{__builtin_amdgcn_perm(0, cb[r], 0x010C000Cu), __builtin_amdgcn_perm(0, cb[r], 0x030C020Cu)};
                if (HP == HP_TEST && test) {
                    // a wave stages the rows of its own part of the tile: lanes that
                    // differ in bits 2 to 5 hold the same four k
                    uint32_t oa[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int r = 0; r < FA; ++r) or_fixed16(ca[r], oa);
#pragma unroll
                    for (int q = 0; q < 4; ++q) oa[q] = row_or<8 | 4>(oa[q]);
                    if ((t & 12) == 0) *(u4v*)&orA[buf][t >> 6][(t >> 4) & 3][sak] = u4v{oa[0], oa[1], oa[2], oa[3]};
#pragma unroll
                    for (int r = 0; r < FB; ++r) {
                        uint32_t ob[4] = {0, 0, 0, 0};
                        or_fixed16(cb[r], ob);
                        const uint32_t v = row_or<8 | 4 | 2 | 1>(ob[0] | ob[1] | ob[2] | ob[3]);
                        // TPB = 32: a k's columns span two 16-lane rows; TPB = 16: one
                        if ((t & 15) == 0) orB[buf][sbk + r * D::RB][D::TPB == 32 ? (t >> 4) & 1 : 0] = v;
                    }
                }
            } else {
                f4 a[FA];
#pragma unroll
                for (int r = 0; r < FA; ++r) a[r] = cast_in4<VI>(ld.ra[r], fi);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    hf v;
#pragma unroll
                    for (int r = 0; r < FA; ++r) v[r] = (_Float16)a[r][q];
                    *(hf*)&As[buf][sak + q][sam] = v;
                }
#pragma unroll
                for (int r = 0; r < FB; ++r) {
                    const f4 b = cast_in4<VI>(ld.rb[r], fi);
                    using hq = typename HVec<4>::T;
                    *(hq*)&Bs[buf][sbk + r * D::RB][sbn] = hq{(_Float16)b.x, (_Float16)b.y, (_Float16)b.z, (_Float16)b.w};
                }
            }
        };
        // bit k: every product of k-step k in this wave's part of the tile is a half
        auto exact_mask = [&](int buf, bool tested) -> uint32_t {
            if (HP != HP_TEST || !tested) return 0u;
            const int k = t & (GK - 1), w = HP == HP_TEST ? t >> 6 : 0;
            const uint32_t a = orA[buf][w][0][k] | orA[buf][w][1][k] | orA[buf][w][2][k] | orA[buf][w][3][k];
            const uint32_t b = orB[buf][HP == HP_TEST ? k : 0][0] | (D::TPB == 32 ? orB[buf][HP == HP_TEST ? k : 0][1] : 0u);
            // lowest bits' exponents sum to >= -24 (each word counts in 2^-16);
            // magnitudes below 2^(ea + eb + 2) <= 2^16.  A zero word passes both.
            const bool ok = __builtin_ctz(a | 0x80000000u) + __builtin_ctz(b | 0x80000000u) >= 8 &&
                            __builtin_clz(a | 1u) + __builtin_clz(b | 1u) >= 16;
            return (uint32_t)__ballot(ok) & 0xFFFFu;
        };
        // one k; EX: every product is a half
        auto step = [&](const hm& av, const hn& bv, auto ex) {
            constexpr bool EX = decltype(ex)::value;
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const h2 a = h2{av[i], av[i]};
                h2 b[TN / 2], p[TN / 2];
#pragma unroll
                for (int h = 0; h < TN / 2; ++h) {
                    b[h] = h2{bv[2 * h], bv[2 * h + 1]};
                    if constexpr (!EX) p[h] = a * b[h];  // rounded to half
                }
                if constexpr (KAHAN) {
                    // each phase over the row's chains in turn, so that no add waits on the one before it
                    h2 y[TN / 2], tt[TN / 2];
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h)
                        y[h] = EX ? __builtin_elementwise_fma(a, b[h], -c[i][h]) : p[h] - c[i][h];
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h) tt[h] = s[i][h] + y[h];
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h) c[i][h] = tt[h] - s[i][h];
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h) {
                        c[i][h] = c[i][h] - y[h];
                        s[i][h] = tt[h];
                    }
                } else {
#pragma unroll
                    for (int h = 0; h < TN / 2; ++h)
                        s[i][h] = EX ? __builtin_elementwise_fma(a, b[h], s[i][h]) : s[i][h] + p[h];
                }
            }
        };
        // NK steps of the staged k-tile from its row kr on, as in k_lp_gemm; bit kk of
        // exact: every product of step kk is a half
        auto steps = [&](auto nk, int buf, int kr, uint32_t exact, bool first) {
            constexpr int NK = decltype(nk)::value;
            hm av = *(const hm*)&As[buf][kr][ty * TM];
            hn bv = *(const hn*)&Bs[buf][kr][tx * TN];
#pragma unroll
            for (int kk = 0; kk < NK; ++kk) {
                hm an = av;
                hn bn = bv;
                if (kk + 1 < NK) {
                    an = *(const hm*)&As[buf][kr + kk + 1][ty * TM];
                    bn = *(const hn*)&Bs[buf][kr + kk + 1][tx * TN];
                }
                __builtin_amdgcn_sched_barrier(0);
                if (HP == HP_FMA || (HP == HP_TEST && ((exact >> kk) & 1u)))
                    step(av, bv, std::true_type{});
                else
                    step(av, bv, std::false_type{});
                if (KAHAN && kk == 0 && first) clear_c();
                av = an;
                bv = bn;
            }
        };
        if (g.K > 0) {
            ld.init(g, m0, n0);
            ld.fetch(g, 0, n0);
            put(0, true);
        }
        if (t == 0) passed[1] = GK;
        __syncthreads();
        int buf = 0;
        int k0 = 0;
        bool tested = HP == HP_TEST;
        for (; k0 + GK <= g.K; k0 += GK, buf ^= 1) {
            const bool more = k0 + GK < g.K;
            if (more) ld.fetch(g, k0 + GK, n0);  // in flight during this tile's math
            const uint32_t exact = exact_mask(buf, tested);
            if constexpr (HP == HP_TEST) {
                const uint32_t before = passed[buf ^ 1];  // written before the last barrier
                if (t == 0) passed[buf] = tested ? __builtin_popcount(exact) : before;
                // the next tile is tested where it pays, and every eighth anyway
                tested = __builtin_amdgcn_readfirstlane((int)before) >= GK / 4 || (k0 / GK) % 8 == 7;
            }
            steps(std::integral_constant<int, GK>{}, buf, 0, exact, k0 == 0);
#pragma unroll
            for (int i = 0; i < TM; ++i)  // as in k_lp_gemm: the chains end before the staging
#pragma unroll
                for (int h = 0; h < TN / 2; ++h) {
                    pin(s[i][h]);
                    if constexpr (KAHAN) pin(c[i][h]);
                }
            if (more) put(buf ^ 1, tested);
            __syncthreads();
        }
        // the rest of K, fewer than GK steps
        int kr = 0;
#pragma unroll 1
        for (; k0 + kr + 8 <= g.K; kr += 8) steps(std::integral_constant<int, 8>{}, buf, kr, 0u, k0 + kr == 0);
#pragma unroll 1
        for (; k0 + kr < g.K; ++kr) steps(std::integral_constant<int, 1>{}, buf, kr, 0u, k0 + kr == 0);
        __syncthreads();  // before another tile is staged
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int64_t m = m0 + ty * TM + i;
            if (m >= g.M) continue;
            float* crow = g.C + m * g.ldc;
            const int64_t n = n0 + tx * TN;
            if (TN >= 4 && n + TN <= g.N) {
#pragma unroll
                for (int h = 0; h + 1 < TN / 2; h += 2)
                    *(f4u*)(crow + n + 2 * h) =
                        f4{(float)s[i][h][0], (float)s[i][h][1], (float)s[i][h + 1][0], (float)s[i][h + 1][1]};
            } else {
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    if (n + j < g.N) crow[n + j] = (float)s[i][j >> 1][j & 1];
            }
        }
    }
}

// ------------------------------------------------------------ launchers

// The grid of k_lp_gemm and k_lp_gemm_h.
inline dim3 gemm_grid(const GemmArgs& g, int gm, int gn) {
    return dim3((unsigned)((g.N + gn - 1) / gn), (unsigned)std::min((g.M + gm - 1) / gm, 65535));
}

// The tiles of k_lp_gemm (outputs per thread).  Measured on MI355X, us, 1-5-2
// inputs: into 1-8-7 plain, then with Kahan's chain into 1-8-7, 1-5-2 and 1-8-23:
//                       4x4   2x2   1x2   1x1 |  4x4   2x2   1x1 |  4x4   2x2   1x1 |  4x4   2x2   1x1
//   4096 x 4096 x 512   469   475   599  1041 | 1806  1788  1705 | 4643  4695  4925 |  634   700  1126
//   1024 x 1024 x 1024  104    76    84   137 |  275   242   226 |  854   655   645 |  235   120   159
//   256 x 1000 x 2048   202    67    52    77 |  541   157   129 | 1695   482   369 |  464   171   100
//   4096 x 4096 x 8      16    27    55    73 |   33    38    76 |   78    91   166 |   23    39   116
//   512 x 512 x 8       3.8   2.9   3.3   3.4 |  4.9   3.1   3.5 |  9.8   5.4   5.6 |  5.3   4.1   5.0
// A plain chain has two to eight VALU instructions per product, so 1 x 1 is
// bound by its two LDS reads per product and 2 x 2 is not; below three 2 x 2
// blocks per CU smaller tiles spread the chains over more waves, down to
// 1 x 1 where even its blocks do not outnumber the CUs.  Kahan's chain hides
// the reads at 1 x 1, whose many waves hide the chain's latency, where its adds
// are one instruction (7 mantissa bits) or bound by fp64; on large products of
// the other classes 1 x 1 costs 5 %, and where an add is the fma alone (1-8-23)
// the reads bind it as they do a plain chain.  A block costs its launch and the
// staging of a whole k-tile however small K is: below K = 64, the largest
// k-tile, large products take 4 x 4 and k-tiles of 16, below 32 the others 2 x 2.
enum GemmTiles { GT_4X4, GT_2X2, GT_1X2, GT_1X1 };

// Outputs computed with tiles of gm x gn, the padding of the edges included.
inline int64_t gemm_padded(const GemmArgs& g, int64_t gm, int64_t gn) {
    return (g.M + gm - 1) / gm * gm * ((g.N + gn - 1) / gn * gn);
}

inline GemmTiles gemm_tiles(const GemmArgs& g, bool kahan, bool exact, bool hides) {
    const auto blocks = [&](int64_t gt) { return gemm_padded(g, gt, gt) / (gt * gt); };
    // whether tiles of gt pad a narrow product to at most `most` times what those of
    // `than` do (2^20 x 4 x 16 into 1-8-7 with Kahan's chain: 219 us at 4 x 4, 96 at
    // 1 x 1; 1-8-23 gains more by 4 x 4, and at the smallest K by 2 x 2, than that costs)
    const auto fits = [&](int64_t gt, int64_t than, double most) {
        return (double)gemm_padded(g, gt, gt) <= most * (double)gemm_padded(g, than, than);
    };
    const bool fit4 = fits(64, kahan ? 16 : 32, exact ? 1.6 : 1.25);
    const bool fit2 = !kahan || fits(32, 16, exact && g.K < 16 ? 2.0 : (g.K < 64 ? 1.25 : 1.05));
    if (exact && blocks(64) >= 512 && (fit4 || !kahan)) return GT_4X4;  // an add is the fma alone
    if (g.K < 64 && blocks(64) >= (g.K < 32 ? 512 : 1024) && fit4) return GT_4X4;
    if (g.K < 32 && fit2) return blocks(16) > 256 ? GT_2X2 : GT_1X1;
    if (kahan) {
        const int64_t least = g.K < 64 || exact ? 768 : (hides ? INT64_MAX : 2048);
        return fit2 && blocks(32) >= least ? GT_2X2 : GT_1X1;
    }
    if (blocks(32) >= 768) return GT_2X2;
    return blocks(16) > 256 ? GT_1X2 : GT_1X1;
}

template <int V, int PM, int VI = -1>
static void launch_gemm(bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi, const FmtK& fa) {
#define APS_GL(K, TM, TN, GK)                                                                                     \
    hipLaunchKernelGGL((k_lp_gemm<V, K, PM, VI, TM, TN, GK>), gemm_grid(g, 16 * TM, 16 * TN), dim3(BLOCK), 0, s, g, \
                       fi, fa)
    // whether Kahan's chain hides the operand reads: 7 mantissa bits, fp64 adds
    constexpr bool hides = PM >= GP_B7_GRID || VT<V>::acc == ACC_F64;
    const GemmTiles tiles = gemm_tiles(g, kahan, VT<V>::acc == ACC_EXACT, hides);
    if (kahan) {
        if (tiles == GT_4X4) APS_GL(true, 4, 4, 16);
        else if (tiles == GT_2X2) APS_GL(true, 2, 2, 32);
        else APS_GL(true, 1, 1, 64);
    } else {
        if (tiles == GT_4X4) APS_GL(false, 4, 4, 16);
        else if (tiles == GT_2X2) APS_GL(false, 2, 2, 32);
        else if (tiles == GT_1X2) APS_GL(false, 1, 2, 64);
        else APS_GL(false, 1, 1, 64);
    }
#undef APS_GL
}

// One accumulator variant V, product mode pm: the modes V can take.
template <int V>
static void launch_gemm_v(int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                          const FmtK& fa) {
    constexpr bool shifted = VT<V>::cls == CLS_TOP || VT<V>::cls == CLS_LOW;
    if (pm == GP_LDEXP) {
        if constexpr (shifted) launch_gemm<V, GP_LDEXP>(kahan, s, g, fi, fa);
    } else if (pm == GP_FIT) {
        if constexpr (shifted && !VT<V>::m0) launch_gemm<V, GP_FIT>(kahan, s, g, fi, fa);
    } else if (pm == GP_GRID) {
        if constexpr (shifted && !VT<V>::m0) {
            if (input_mode_is(VI_E5M2, fi))
                launch_gemm<V, GP_GRID, VI_E5M2>(kahan, s, g, fi, fa);
            else if (input_mode_is(VI_E4M3, fi))
                launch_gemm<V, GP_GRID, VI_E4M3>(kahan, s, g, fi, fa);
            else
                launch_gemm<V, GP_GRID>(kahan, s, g, fi, fa);
        }
    } else if (pm == GP_EXACT) {
        if constexpr (!VT<V>::m0) launch_gemm<V, GP_EXACT>(kahan, s, g, fi, fa);
    } else if (pm == GP_FMA) {
        if constexpr (!VT<V>::m0 && VT<V>::acc != ACC_F64) launch_gemm<V, GP_FMA>(kahan, s, g, fi, fa);
    } else {
        launch_gemm<V, GP_SCALED>(kahan, s, g, fi, fa);
    }
}

// By accumulator class (variants INT, TOP, LOW), one file each.
void launch_gemm_int(int variant, int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                     const FmtK& fa);
void launch_gemm_top(int variant, int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                     const FmtK& fa);
void launch_gemm_low(int variant, int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi,
                     const FmtK& fa);
// Accumulators of 7 mantissa bits, pm one of GP_B7_*.
void launch_gemm_b7(int pm, bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi, const FmtK& fa);
// The IEEE half accumulator; false where no kernel takes the input's class.
bool launch_gemm_half(bool kahan, hipStream_t s, const GemmArgs& g, const FmtK& fi);

}  // namespace aps
