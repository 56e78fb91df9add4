// aps_codes.hip -- the W-worker rounded sum over packed codes, the form in
// which workers would exchange the cast gradients (Algorithm 1's SUM
// all-reduce of the cast gradients; Sec. 5).
#include "aps_common.hpp"

namespace aps {

// ================================================ K4c: reduce of packed codes

struct CodesArgs {
    const uint8_t* __restrict__ codes;  // W rows of packed codes
    float* __restrict__ out;
    uint8_t* __restrict__ codes_out;
    int64_t row_bytes;  // bytes per code row (a multiple of 16)
    int32_t W;
    uint32_t flags;
};

// Per-element scale exponents for N consecutive elements from j.
template <int N>
__device__ __forceinline__ void elem_scales_n(const Layers& ly, const ChunkInfo& ci, int64_t j, int32_t* ft) {
    int li = ci.i0;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        while (li < ci.i1 && ly.offsets[li + 1] <= j + e) ++li;
        ft[e] = ly.scale_exp ? clamp_exp(ly.scale_exp[li]) : 0;
    }
}

// Rows per register set.  A thread's sums and decoded codes take 32 (nibbles:
// 64) registers, so two sets of 4 rows leave two waves per SIMD where sets
// of 2 leave four (ResNet-50, W = 8, sum and decode: 1-3-0 183 -> 121 us,
// 1-4-3 94 -> 89, 1-5-2 79 -> 78; W = 256 the same).
constexpr int CODES_UNROLL = 2;

// The hardware form a palette entry's codes of class CC take.
__host__ __device__ __forceinline__ int hw_of_codes(const FmtK& f, int cc) {
    return cc == 1 && (f.hw == HW_E5M2 || f.hw == HW_E4M3) ? f.hw : (cc == 2 && f.hw == HW_HALF ? f.hw : HW_NONE);
}

// Code e (0..EPT-1) of a thread's 16-byte slice.
template <int CC>
__device__ __forceinline__ uint32_t slice_code(const f4& v, int e) {
    const uint32_t w[4] = {f2u(v.x), f2u(v.y), f2u(v.z), f2u(v.w)};
    if constexpr (CC == 0) return (w[e >> 3] >> ((e & 7) * 4)) & 15u;
    else if constexpr (CC == 1) return (w[e >> 2] >> ((e & 3) * 8)) & 255u;
    else return (w[e >> 1] >> ((e & 1) * 16)) & 0xFFFFu;
}

// The W-worker rounded sum of already scaled and cast gradients given as
// packed codes (the low-precision values the workers exchange).  A thread
// owns the codes in 16 bytes of each row: 32 nibble, 16 byte or 8 uint16
// codes.  Three formats run on the hardware's conversions (HW):
//   1-5-2   decoded two codes per instruction and every sum rounded by the
//           conversion to E5M2 and back (native values): 2.5 VALU
//           instructions per code;
//   1-4-3   decoded by the conversion from E4M3 and a multiply into the
//           working domain, where overflow is fp32's;
//   1-5-10  the codes are halves: one packed half add per two codes.
// Other codes of up to 8 bits decode through a table of working-domain values
// in LDS, whose random reads (about 7 clocks per wave and code with bank
// conflicts) weigh as much as the HBM reads; other 16-bit codes decode
// arithmetically.  ResNet-50, W = 8, the sum to codes and their decode: 1-5-2
// 104 -> 75 us, 1-4-3 107 -> 85, 1-5-10 367 -> 112; W = 256 1-5-2 1197 -> 1069.
template <int V, int CC, int HW>
__global__ __launch_bounds__(BLOCK) void k_sim_reduce_codes(CodesArgs a, Layers ly, Pal pal) {
    constexpr int EPT = CC == 0 ? 32 : (CC == 1 ? 16 : 8);
    constexpr int64_t CHC = (int64_t)BLOCK * EPT;
    constexpr bool TABLE = CC < 2 && HW == HW_NONE;
    constexpr bool NATIVE = HW == HW_E5M2 || HW == HW_HALF;  // s holds native values, not working-domain ones
    __shared__ float lut[TABLE ? 256 : 1];
    // each wave's fp32 outputs pass through its own LDS slots, so that they
    // leave in stores of consecutive 16-byte pieces per lane (a lane's EPT
    // outputs written as EPT/4 stores 4*EPT bytes apart wrote up to 1.7x
    // the output's bytes to HBM)
    __shared__ __align__(16) float ostage[BLOCK * EPT];
    int lut_pidx = -1;
    const int64_t nchunks = (ly.n + CHC - 1) / CHC;
    int64_t cb, ce;
    block_range(nchunks, cb, ce);
    LayerCur cur{-1, 0};
    for (int64_t c = cb; c < ce; ++c) {
        const int64_t start = c * CHC;
        const int64_t end = min(start + CHC, ly.n);
        const ChunkInfo ci = chunk_layers(ly, start, end, cur);
        if (ci.mixed) continue;
        const FmtK& f = pal.f[ci.pidx];
        if (f.variant != V || hw_of_codes(f, CC) != HW) continue;
        if constexpr (TABLE) {
            if (ci.pidx != lut_pidx) {  // uniform
                __syncthreads();
                for (int t = threadIdx.x; t < (CC == 0 ? 16 : 256); t += BLOCK)
                    lut[t] = __builtin_amdgcn_ldexpf(decode((uint32_t)t, f), f.k);
                __syncthreads();
                lut_pidx = ci.pidx;
            }
        }
        const int64_t j = start + (int64_t)threadIdx.x * EPT;
        if (j >= end) continue;
        const uint8_t* p = a.codes + code_byte(j, CC);
        const int64_t rb = a.row_bytes;
        float s[EPT];
        h2 sh[4];  // HW_HALF: the sums, two per register
        uint32_t bad = 0;
        uint32_t nan[4] = {0, 0, 0, 0};  // HW_E4M3: the top bit of byte e: a code of element e was a NaN
        // the values of a thread's codes in one row
        auto decode_row = [&](const f4& v, float (&d)[EPT]) {
            if constexpr (HW == HW_E5M2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) decode4_e5m2(f2u(v[q]), d + 4 * q);
            } else if constexpr (HW == HW_E4M3) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    decode4_e4m3(f2u(v[q]), d + 4 * q);
                    nan[q] |= nan_bytes_e4m3(f2u(v[q]));  // a NaN stays to the chain's end
                }
            } else {
#pragma unroll
                for (int e = 0; e < EPT; ++e) {
                    const uint32_t code = slice_code<CC>(v, e);
                    if constexpr (TABLE) d[e] = lut[code];
                    else d[e] = __builtin_amdgcn_ldexpf(decode(code, f), f.k);
                }
            }
        };
        stream_rows<CODES_UNROLL>(
            a.W, [&](int r) { return ld4((const float*)(p + (int64_t)r * rb)); }, [&]() {},
            [&](const f4& v) {
                if constexpr (HW == HW_HALF) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) sh[q] = __builtin_bit_cast(h2, f2u(v[q]));
                } else {
                    decode_row(v, s);
                }
            },
            [&](const f4& v, bool valid) {
                if (!valid) return;
                if constexpr (HW == HW_HALF) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) sh[q] = sh[q] + __builtin_bit_cast(h2, f2u(v[q]));  // rounded to half
                    return;
                }
                // all of the row's values first, so the table reads' latencies
                // overlap instead of each add waiting for its own read
                float d[EPT];
                decode_row(v, d);
                if constexpr (TABLE) __builtin_amdgcn_sched_barrier(0);
                if constexpr (HW == HW_E5M2) {
#pragma unroll
                    for (int e = 0; e < EPT; e += 2) round2_e5m2(s[e] + d[e], s[e + 1] + d[e + 1], s[e], s[e + 1]);
                } else {
#pragma unroll
                    for (int e = 0; e < EPT; ++e) {
                        bool b = false;
                        s[e] = accum<V>(s[e], d[e], f, b);
                        if constexpr (VT<V>::m0) bad |= (uint32_t)b << e;
                    }
                }
            });
        if constexpr (HW == HW_HALF) {
#pragma unroll
            for (int e = 0; e < EPT; ++e) s[e] = (float)sh[e >> 1][e & 1];
        }
        if constexpr (HW == HW_E4M3) {
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                s[e] = (nan[e >> 2] >> (8 * (e & 3) + 7)) & 1u ? __builtin_nanf("") : s[e];
        }
        // output exponents, per element when the chunk crosses layers
        const int32_t fdom = ((a.flags & APS_OUTPUT_SCALED) ? 0 : 1);
        const int32_t k = NATIVE ? 0 : f.k;
        int32_t ft[EPT];
        if (ci.i0 == ci.i1) {
            const int32_t t = ly.scale_exp ? clamp_exp(cld(ly.scale_exp, ci.i0)) : 0;
#pragma unroll
            for (int e = 0; e < EPT; ++e) ft[e] = t;
        } else {
            elem_scales_n<EPT>(ly, ci, j, ft);
        }
        float o[EPT];
        uint32_t cw[4] = {0, 0, 0, 0};
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const float se = VT<V>::m0 ? (((bad >> e) & 1u) ? __builtin_nanf("") : s[e]) : s[e];
            o[e] = __builtin_amdgcn_ldexpf(se, -(fdom * ft[e] + k));
            if constexpr (HW == HW_NONE) {
                if (a.codes_out) {
                    const uint32_t cd = encode(__builtin_amdgcn_ldexpf(se, -f.k), f);
                    if constexpr (CC == 0) cw[e >> 3] |= (cd & 15u) << ((e & 7) * 4);
                    else if constexpr (CC == 1) cw[e >> 2] |= (cd & 255u) << ((e & 3) * 8);
                    else cw[e >> 1] |= (cd & 0xFFFFu) << ((e & 1) * 16);
                }
            }
        }
        if (HW == HW_E5M2 && a.codes_out) {
#pragma unroll
            for (int q = 0; q < 4; ++q) cw[q] = encode4_e5m2(s[4 * q], s[4 * q + 1], s[4 * q + 2], s[4 * q + 3]);
        }
        if (HW == HW_E4M3 && a.codes_out) {
            constexpr float ik = 0x1p-120f;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                cw[q] = encode4_e4m3(s[4 * q] * ik, s[4 * q + 1] * ik, s[4 * q + 2] * ik, s[4 * q + 3] * ik);
        }
        if (HW == HW_HALF && a.codes_out) {
#pragma unroll
            for (int q = 0; q < 4; ++q) cw[q] = canonical2_half(__builtin_bit_cast(uint32_t, sh[q]));
        }
        const int lane = threadIdx.x & 63;
        const int64_t wbase = j - (int64_t)lane * EPT;  // the wave's first element
        if (wbase + 64 * EPT <= end) {
            // the whole wave is inside the gradient: every lane is here
            if (a.out) {
                float* wbuf = ostage + (threadIdx.x - lane) * EPT;
#pragma unroll
                for (int q = 0; q < EPT / 4; ++q) {
                    const f4 v = {o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]};
                    *(f4*)(wbuf + lane * EPT + 4 * q) = v;
                }
                wave_lds_sync();
#pragma unroll
                for (int q = 0; q < EPT / 4; ++q) {
                    const f4 v = *(const f4*)(wbuf + 4 * lane + 256 * q);
                    __builtin_nontemporal_store(v, (f4*)(a.out + wbase + 4 * lane + 256 * q));
                }
                wave_lds_sync();
            }
            if (a.codes_out) {
                const u4v v = {cw[0], cw[1], cw[2], cw[3]};
                __builtin_nontemporal_store(v, (u4v*)(a.codes_out + code_byte(j, CC)));
            }
        } else {
            // the wave reaches the ragged end of the gradient: element by element
            for (int e = 0; e < EPT && j + e < end; ++e) {
                if (a.out) a.out[j + e] = o[e];
                if (a.codes_out) {
                    const int64_t jj = j + e;
                    if constexpr (CC == 0) {
                        const uint32_t cd = (cw[e >> 3] >> ((e & 7) * 4)) & 15u;
                        uint8_t* pb = a.codes_out + (jj >> 1);
                        const int sh = (int)(jj & 1) * 4;
                        *pb = (uint8_t)((*pb & ~(15u << sh)) | (cd << sh));
                    } else if constexpr (CC == 1) {
                        a.codes_out[jj] = (uint8_t)(cw[e >> 2] >> ((e & 3) * 8));
                    } else {
                        *(uint16_t*)(a.codes_out + 2 * jj) = (uint16_t)(cw[e >> 1] >> ((e & 1) * 16));
                    }
                }
            }
        }
    }
}

// Mixed-format chunks of the codes reduce: element pairs per thread, any variant.
template <int V>
__device__ float reduce_codes_elem(const CodesArgs& a, const FmtK& f, int cc, int64_t j) {
    bool bad = false;
    const int64_t cb = code_byte(j, cc);
    auto get = [&](int w) -> float {
        const uint8_t* row = a.codes + (int64_t)w * a.row_bytes;
        uint32_t code;
        if (cc == 0)
            code = (row[cb] >> ((j & 1) * 4)) & 15u;
        else if (cc == 1)
            code = row[cb];
        else
            code = *(const uint16_t*)(row + cb);
        return __builtin_amdgcn_ldexpf(decode(code, f), f.k);
    };
    float s = get(0);
    for (int w = 1; w < a.W; ++w) s = accum<V>(s, get(w), f, bad);
    return finish<V>(s, bad);
}

__device__ float reduce_codes_any(const CodesArgs& a, const FmtK& f, int cc, int64_t j) {
    switch (f.variant) {
        case V_INT_F32: return reduce_codes_elem<V_INT_F32>(a, f, cc, j);
        case V_INT_F64: return reduce_codes_elem<V_INT_F64>(a, f, cc, j);
        case V_INT_EXACT: return reduce_codes_elem<V_INT_EXACT>(a, f, cc, j);
        case V_INT_M0: return reduce_codes_elem<V_INT_M0>(a, f, cc, j);
        case V_TOP_F32: return reduce_codes_elem<V_TOP_F32>(a, f, cc, j);
        case V_TOP_F64: return reduce_codes_elem<V_TOP_F64>(a, f, cc, j);
        case V_TOP_M0: return reduce_codes_elem<V_TOP_M0>(a, f, cc, j);
        case V_LOW_F32: return reduce_codes_elem<V_LOW_F32>(a, f, cc, j);
        case V_LOW_F64: return reduce_codes_elem<V_LOW_F64>(a, f, cc, j);
        case V_GEN: return reduce_codes_elem<V_GEN>(a, f, cc, j);
        default: return reduce_codes_elem<V_LOW_M0>(a, f, cc, j);
    }
}

// One block per layer boundary; the chunk (of the codes reduce's chunk size)
// owning the first boundary strictly inside it, when it mixes palette entries.
template <int CC>
__global__ __launch_bounds__(BLOCK) void k_sim_reduce_codes_mixed(CodesArgs a, Layers ly, Pal pal) {
    constexpr int64_t CHC = (int64_t)BLOCK * (CC == 0 ? 32 : (CC == 1 ? 16 : 8));
    __shared__ FmtK spal[APS_MAX_FORMATS];
    pal_to_lds(pal, spal);
    const int b = blockIdx.x;
    if (b < 1 || b >= ly.L) return;
    const int64_t pb = cld(ly.offsets, b);
    if (pb <= 0 || pb >= ly.n || pb % CHC == 0) return;
    const int64_t start = pb / CHC * CHC;
    const int64_t end = min(start + CHC, ly.n);
    if (cld(ly.offsets, b - 1) > start) return;
    if (!chunk_layers(ly, start, end).mixed) return;
    for (int64_t j0 = start + 2 * (int64_t)threadIdx.x; j0 < end; j0 += 2 * BLOCK) {
        uint32_t cd[2] = {0, 0};
        for (int e = 0; e < 2; ++e) {
            const int64_t j = j0 + e;
            if (j >= end) break;
            const int li = find_layer(ly.offsets, ly.L, j, 0);
            const FmtK& f = spal[ly.fmt_idx[li]];
            const int32_t ft = ly.scale_exp ? clamp_exp(ly.scale_exp[li]) : 0;
            const float sv = reduce_codes_any(a, f, CC, j);
            const int fd = (a.flags & APS_OUTPUT_SCALED) ? 0 : ft;
            if (a.out) a.out[j] = __builtin_amdgcn_ldexpf(sv, -(fd + f.k));
            cd[e] = encode(__builtin_amdgcn_ldexpf(sv, -f.k), f);
            if (a.codes_out && CC != 0) put_code(a.codes_out, j, cd[e], CC);
        }
        if (a.codes_out && CC == 0) {
            uint8_t* q = a.codes_out + (j0 >> 1);
            *q = (j0 + 1 < end) ? (uint8_t)((cd[0] & 15u) | ((cd[1] & 15u) << 4))
                                : (uint8_t)((*q & 0xF0u) | (cd[0] & 15u));
        }
    }
}

}  // namespace aps

using namespace aps;

extern "C" int aps_sim_reduce_codes(const void* codes, int32_t W, int64_t ld, int64_t n, const int64_t* offsets,
                                    int32_t L, const int32_t* scale_exp, const aps_format* fmts, int32_t n_fmts,
                                    const uint8_t* fmt_idx, uint32_t flags, float* out, void* codes_out,
                                    void* stream) {
    if (!codes || !offsets) return APS_ERR_NULL;
    if (W < 1 || W > APS_MAX_WORKERS || L < 1 || n < 0 || n > APS_MAX_ELEMS || ld < n) return APS_ERR_SIZE;
    if (!out && !codes_out && n > 0) return APS_ERR_NULL;
    if (flags & ~APS_OUTPUT_SCALED) return APS_ERR_UNSUPPORTED;
    Pal pal;
    int ccls = 0;
    int st = check_palette(fmts, n_fmts, pal, &ccls);
    if (st != APS_OK) return st;
    if (ccls < 0 || ccls > 2) return APS_ERR_UNSUPPORTED;
    const int64_t row_bytes = code_byte(ld, ccls);
    if (!aligned16(codes) || (row_bytes & 15) || (out && !aligned16(out)) || (codes_out && !aligned16(codes_out)))
        return APS_ERR_ALIGN;
    if (n == 0) return APS_OK;
    hipStream_t s = (hipStream_t)stream;
    Layers ly{offsets, fmt_idx, scale_exp, n, L, n_fmts};
    CodesArgs a{(const uint8_t*)codes, out, (uint8_t*)codes_out, row_bytes, W, flags};
    const int64_t ept = ccls == 0 ? 32 : (ccls == 1 ? 16 : 8);
    const int64_t nchunks = (n + BLOCK * ept - 1) / (BLOCK * ept);
    // a block per chunk up to 64 per CU: blocks of a chunk or two balance
    // better than 16 per CU (ResNet-50, W = 64: 1-5-2 334 -> 307 us, 1-5-10
    // 639 -> 579 us; W = 8 the same)
    const dim3 grid((unsigned)grid_for(nchunks, 64));
    // (16-bit codes decode so slowly without the hardware that a large set is
    // worth 1-5-10's own launch: 1-5-10 and 1-5-7 in turn, one launch and two, us:
    // 25.6 M W = 8 183 and 167, 3 M W = 64 276 and 262, 0.3 M W = 256 785 and 820)
    if (ccls < 2 || (int64_t)W * n < ((int64_t)1 << 27))
        one_form_per_variant(
            pal, n_fmts, [](const FmtK& f) { return f.variant; }, [&](const FmtK& f) { return hw_of_codes(f, ccls); });
    unsigned vm = 0, hm = 0;  // variants of the entries without, and forms of those with, hardware codes
    for (int i = 0; i < n_fmts; ++i) {
        const int hw = hw_of_codes(pal.f[i], ccls);
        if (hw) hm |= 1u << hw;
        else vm |= 1u << pal.f[i].variant;
    }
#define APS_C(v, c, h) hipLaunchKernelGGL((k_sim_reduce_codes<v, c, h>), grid, dim3(BLOCK), 0, s, a, ly, pal)
    if (hm & (1u << HW_E5M2)) APS_C(V_TOP_F32, 1, HW_E5M2);
    if (hm & (1u << HW_E4M3)) APS_C(V_LOW_F32, 1, HW_E4M3);
    if (hm & (1u << HW_HALF)) APS_C(V_TOP_F32, 2, HW_HALF);
#define APS_LAUNCH_C(v)                      \
    if (vm & (1u << (v))) {                  \
        if (ccls == 0) APS_C(v, 0, HW_NONE); \
        if (ccls == 1) APS_C(v, 1, HW_NONE); \
        if (ccls == 2) APS_C(v, 2, HW_NONE); \
    }
    APS_FOR_VARIANTS(APS_LAUNCH_C)
#undef APS_LAUNCH_C
#undef APS_C
    if (fmt_idx && n_fmts > 1 && L > 1) {
        if (ccls == 0) hipLaunchKernelGGL(k_sim_reduce_codes_mixed<0>, dim3((unsigned)L), dim3(BLOCK), 0, s, a, ly, pal);
        if (ccls == 1) hipLaunchKernelGGL(k_sim_reduce_codes_mixed<1>, dim3((unsigned)L), dim3(BLOCK), 0, s, a, ly, pal);
        if (ccls == 2) hipLaunchKernelGGL(k_sim_reduce_codes_mixed<2>, dim3((unsigned)L), dim3(BLOCK), 0, s, a, ly, pal);
    }
    return launched();
}
