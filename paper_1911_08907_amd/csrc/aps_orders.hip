// aps_orders.hip -- the W-worker rounded sum in the order of the
// hierarchical all-reduce of Sec. 4.2 (groups, ring over the masters), with
// the plain or Kahan low-precision accumulator of Sec. 5.
#include <type_traits>

#include "aps_common.hpp"

namespace aps {

// ======================================= K4x: summation orders, Kahan

struct Order {
    int32_t log2k;  // group size k = 2^log2k
    int32_t ng;     // number of groups W / k
};

// Worker of the r-th add for an element of ring segment seg: the groups in
// master order seg, seg+1, ... (mod ng), each in worker order.
__device__ __forceinline__ int order_row(int r, int seg, const Order& od) {
    int g = seg + (r >> od.log2k);
    if (g >= od.ng) g -= od.ng;
    return (g << od.log2k) + (r & ((1 << od.log2k) - 1));
}

// The chains of a thread's 4 elements: how a value is cast, and one add of a
// chain (plain, or Kahan's).  In general, in the variant's working domain; for
// 1-5-2 and 1-5-10 on native values by the hardware: a cast or a rounded add
// of 1-5-2 is the conversion to E5M2 and back (two values each), one
// instruction per value beside the add where the general form takes three to
// nine, and 1-5-10 is the packed half arithmetic itself.
template <int V, int HW, bool KAHAN>
struct Chain4 {
    float s[4], c[4];
    __device__ __forceinline__ static int domain(const FmtK& f) { return HW == HW_NONE ? f.k : 0; }
    __device__ __forceinline__ void cast(const f4& x, const int F[4], const FmtK& f, float q[4],
                                                bool (&flag)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (HW == HW_NONE) q[e] = quant<V>(x[e], F[e], f, flag[e]);
            else q[e] = __builtin_amdgcn_ldexpf(x[e], F[e]);
        }
        if constexpr (HW == HW_E5M2) {
            round2_e5m2(q[0], q[1], q[0], q[1]);
            round2_e5m2(q[2], q[3], q[2], q[3]);
        }
    }
    // the first value of a chain
    __device__ __forceinline__ void start(const float q[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            s[e] = q[e];
            c[e] = 0.0f;
        }
    }
    // q joins the chain; `flag` as chain_step's `bad`
    __device__ __forceinline__ void add(const float q[4], const FmtK& f, bool (&flag)[4]) {
        if constexpr (HW == HW_E5M2) {
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                if constexpr (KAHAN) {
                    float y0, y1, t0, t1, u0, u1;
                    round2_e5m2(q[e] - c[e], q[e + 1] - c[e + 1], y0, y1);
                    round2_e5m2(s[e] + y0, s[e + 1] + y1, t0, t1);
                    round2_e5m2(t0 - s[e], t1 - s[e + 1], u0, u1);
                    round2_e5m2(u0 - y0, u1 - y1, c[e], c[e + 1]);
                    s[e] = t0;
                    s[e + 1] = t1;
                } else {
                    round2_e5m2(s[e] + q[e], s[e + 1] + q[e + 1], s[e], s[e + 1]);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) chain_step<V, KAHAN>(s[e], c[e], q[e], f, flag[e]);
        }
    }
};

// 1-5-10: the same interface on halves, two elements per register.
template <int V, bool KAHAN>
struct Chain4<V, HW_HALF, KAHAN> {
    h2 s[2], c[2];
    __device__ __forceinline__ static int domain(const FmtK&) { return 0; }
    __device__ __forceinline__ void cast(const f4& x, const int F[4], const FmtK&, h2 q[2], bool (&)[4]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            q[h] = h2{(_Float16)__builtin_amdgcn_ldexpf(x[2 * h], F[2 * h]),
                      (_Float16)__builtin_amdgcn_ldexpf(x[2 * h + 1], F[2 * h + 1])};
    }
    __device__ __forceinline__ void start(const h2 q[2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s[h] = q[h];
            c[h] = h2{0, 0};
        }
    }
    __device__ __forceinline__ void add(const h2 q[2], const FmtK&, bool (&)[4]) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (KAHAN) {
                const h2 y = q[h] - c[h];
                const h2 t = s[h] + y;
                c[h] = (t - s[h]) - y;
                s[h] = t;
            } else {
                s[h] = s[h] + q[h];
            }
        }
    }
};

template <int V, int HW, bool KAHAN>
__device__ __forceinline__ void reduce_vec_ex(const ReduceArgs& a, const FmtK& f, int64_t j, int64_t lim,
                                              const int32_t ft[4], int seg, const Order& od, PendingOut& pd) {
    using C = Chain4<V, HW, KAHAN>;
    using Q = std::conditional_t<HW == HW_HALF, h2[2], float[4]>;
    const bool inq = a.flags & APS_INPUT_QUANTIZED;
    const bool outs = a.flags & APS_OUTPUT_SCALED;
    const int k = C::domain(f);
    int F[4], Fo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        F[e] = (inq ? 0 : ft[e]) + k;
        Fo[e] = -((outs ? 0 : ft[e]) + k);
    }
    C S, T;  // the group's chain, the ring's
    bool bad[4] = {false, false, false, false};
    const float* p = a.G + j;
    const int64_t ld = a.ld;
    const int kg = 1 << od.log2k;
    int r = 1;  // index of the next add in the order
    auto zero = [](Q& q) {
        for (auto& v : q) v = std::remove_reference_t<decltype(v)>{};
    };
    stream_rows(
        a.W, [&](int rr) { return ld4(p + (int64_t)order_row(rr, seg, od) * ld); }, [&]() { flush_out(a, pd); },
        [&](const f4& x) {
            Q q;
            S.cast(x, F, f, q, bad);
            S.start(q);  // master of the first group
            zero(q);
            T.start(q);
        },
        [&](const f4& x, bool valid) {
            if (valid) {
                Q q;
                S.cast(x, F, f, q, bad);
                if ((r & (kg - 1)) == 0) {
                    // a new group starts: fold the finished group sum into the ring
                    if (r == kg) T.start(S.s);
                    else T.add(S.s, f, bad);
                    S.start(q);
                } else {
                    S.add(q, f, bad);
                }
            }
            ++r;
        });
    if (od.ng > 1) {
        T.add(S.s, f, bad);
    } else {
        T.start(S.s);
    }
    float s[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (HW == HW_HALF) s[e] = (float)T.s[e >> 1][e & 1];
        else s[e] = finish<V>(T.s[e], bad[e]);
    }
    pd.o.x = __builtin_amdgcn_ldexpf(s[0], Fo[0]);
    pd.o.y = __builtin_amdgcn_ldexpf(s[1], Fo[1]);
    pd.o.z = __builtin_amdgcn_ldexpf(s[2], Fo[2]);
    pd.o.w = __builtin_amdgcn_ldexpf(s[3], Fo[3]);
    if (a.codes) {
#pragma unroll
        for (int e = 0; e < 4; ++e) pd.c[e] = encode(__builtin_amdgcn_ldexpf(s[e], -k), f);
    }
    pd.j = j;
    pd.lim = lim;
    pd.valid = true;
}

__device__ __forceinline__ int64_t ring_segment(int64_t j, int64_t n, int ng) { return j * ng / n; }

// The hardware form of an entry's chains.
__host__ __device__ __forceinline__ int hw_of_chain(const FmtK& f) { return f.hw == HW_E4M3 ? HW_NONE : f.hw; }

// Elements from `at` on up to the end of their ring segment.
struct Span {
    int64_t at, hi;
    int seg;
};

// Segment seg holds the elements i with floor(i * ng / n) = seg.
__device__ __forceinline__ int64_t segment_end(int seg, int64_t n, int ng) { return ((seg + (int64_t)1) * n + ng - 1) / ng; }

// The chunk that cross block b of ncross takes and its first segment's part
// (from the chunk's start on), or false: with fewer segment boundaries than
// chunks one block per boundary (that of the first boundary inside a chunk
// owns it), else one per chunk.
__device__ __forceinline__ bool cross_chunk(int b, int ncross, int64_t n, const Order& od, int64_t& c, Span& sp) {
    if (ncross < od.ng - 1) {
        c = b;
        sp.at = c * CH;
        sp.seg = (int)ring_segment(sp.at, n, od.ng);
        sp.hi = segment_end(sp.seg, n, od.ng);
        return sp.hi < min(sp.at + CH, n);
    }
    sp.seg = b;
    sp.hi = segment_end(b, n, od.ng);  // boundary: first element of segment b + 1
    c = sp.hi / CH;
    sp.at = c * CH;
    if (sp.hi >= n || sp.hi == sp.at) return false;                // at a chunk edge: nothing crosses
    return b == 0 || segment_end(b - 1, n, od.ng) <= sp.at;  // else an earlier boundary owns it
}

// Stores those of a thread's 4 finished outputs that lie in [lo, hi).  A
// thread owns both nibbles of its code bytes, so the read-modify-writes of a
// byte split between segments come in program order.
__device__ __forceinline__ void store_part(const ReduceArgs& a, const PendingOut& pd, int64_t lo, int64_t hi) {
    const float o[4] = {pd.o.x, pd.o.y, pd.o.z, pd.o.w};
    int32_t j = (int32_t)pd.j;  // addresses from here on, not held over the walk (25 registers)
    asm volatile("" : "+v"(j));
    for (int e = 0; e < 4; ++e) {
        const int64_t jj = (int64_t)j + e;
        if (jj < lo || jj >= hi) continue;
        if (a.out) a.out[jj] = o[e];
        if (!a.codes) continue;
        if (a.code_cls == 0) {
            uint8_t* pb = a.codes + (jj >> 1);
            *pb = (jj & 1) ? (uint8_t)((*pb & 0x0Fu) | ((pd.c[e] & 15u) << 4)) : (uint8_t)((*pb & 0xF0u) | (pd.c[e] & 15u));
        } else {
            put_code(a.codes, jj, pd.c[e], a.code_cls);
        }
    }
}

// Which chunks a copy of the walk below takes.
enum ExChunks { EX_WHOLE = 0, EX_CROSS = 1, EX_BOTH = 2 };

// Chunk c: a walk of the rows, or where it crosses ring segments (sp: its
// first segment's part) one per segment with an element in the chunk, whose
// elements are stored after it.
template <int V, int HW, bool KAHAN, int WHICH>
__device__ __forceinline__ void ex_chunk(const ReduceArgs& a, const Layers& ly, const Pal& pal, const Order& od, int64_t c,
                                         Span sp, LayerCur& cur, PendingOut& pd) {
    const int64_t start = c * CH;
    const int64_t end = min(start + CH, ly.n);
    const ChunkInfo ci = chunk_layers(ly, start, end, cur);
    if (ci.mixed) return;  // k_sim_reduce_ex_slow
    const FmtK& f = pal.f[ci.pidx];
    if (f.variant != V || hw_of_chain(f) != HW) return;
    const int64_t j = start + (int64_t)threadIdx.x * VEC;
    if (j >= end) return;
    int32_t ft[4];
    if (ci.i0 == ci.i1) {
        const int32_t t = ly.scale_exp ? clamp_exp(cld(ly.scale_exp, ci.i0)) : 0;
        ft[0] = ft[1] = ft[2] = ft[3] = t;
    } else {
        elem_scales(ly, ci, j, ft);
    }
    if constexpr (WHICH == EX_WHOLE) {
        reduce_vec_ex<V, HW, KAHAN>(a, f, j, end, ft, sp.seg, od, pd);
        return;
    }
    for (;;) {
        reduce_vec_ex<V, HW, KAHAN>(a, f, j, end, ft, sp.seg, od, pd);
        if (sp.at == start && sp.hi >= end) return;  // a whole chunk
        store_part(a, pd, sp.at, min(sp.hi, end));
        pd.valid = false;
        if (sp.hi >= end) return;
        // segments without an element (more segments than elements) take no
        // walk: the next one is that of the first element not yet stored
        sp.at = sp.hi;
        sp.seg = od.ng <= ly.n ? sp.seg + 1 : (int)ring_segment(sp.at, ly.n, od.ng);
        sp.hi = segment_end(sp.seg, ly.n, od.ng);
    }
}

constexpr bool ex_m0(int V) { return V == V_INT_M0 || V == V_TOP_M0 || V == V_LOW_M0; }

// Waves per SIMD asked of an instance: four (at most 128 registers) where that
// costs no scratch or little: 1-5-2 and the fp32 chains fit, Kahan's chains of
// the GEN formats spill 7 registers (12 beside a crossing copy) and wide ones
// (fp64 adds) 17 beside one, and gain all the same.  Without a crossing copy the
// wide ones are left to the compiler (137 registers), as are Kahan's m = 0
// chains (152 to 154), three waves each: held to 128 the latter spill 46, in
// the row walk too.
constexpr int ex_waves(int V, bool KAHAN, bool CROSS) {
    const bool wide = V == V_INT_F64 || V == V_TOP_F64 || V == V_LOW_F64;
    return KAHAN && (ex_m0(V) || (wide && !CROSS)) ? 1 : 4;
}

// CROSS: the first `ncross` blocks take the chunks that cross ring segments,
// one each, whose lone walks, two or more per chunk and bound by latency, so
// run beside the other blocks' instead of after them (ResNet-50 W = 64: 45 us
// of 1190).  They have a copy of the walk to themselves, so that the other
// blocks' keeps its registers, but for Kahan's m = 0 chains, where one copy
// serves both.  Measured on MI355X, us, a launch of the crossing chunks after
// the others and this one: ResNet-50 W = 64 k = 16 Kahan 1-5-2 1216 and 1160,
// 1-3-0 1349 and 1260; W = 8 k = 2 plain 187 and 175 to 179; W = 2 ring plain
// 1-3-0 98 and 87; ResNet-20 W = 8 ring 16 to 20 and 8 to 11.
template <int V, int HW, bool KAHAN, bool CROSS>
__global__ __launch_bounds__(BLOCK, ex_waves(V, KAHAN, CROSS)) void k_sim_reduce_ex(ReduceArgs a, Layers ly, Pal pal,
                                                                                   Order od, int ncross) {
    constexpr bool ONE = ex_m0(V) && KAHAN;
    LayerCur cur{-1, 0};
    PendingOut pd;
    pd.valid = false;
    const int64_t nchunks = (ly.n + CH - 1) / CH;
    const int64_t nb = (int64_t)gridDim.x - ncross, b = (int64_t)blockIdx.x - ncross;
    int64_t c, ce;
    Span sp;
    const bool cross = CROSS && b < 0;
    if (cross) {
        if (!cross_chunk(blockIdx.x, ncross, ly.n, od, c, sp)) return;
        ce = c + 1;
        if constexpr (!ONE) {
            ex_chunk<V, HW, KAHAN, EX_CROSS>(a, ly, pal, od, c, sp, cur, pd);
            return;
        }
    } else {
        c = nchunks * b / nb;
        ce = nchunks * (b + 1) / nb;
    }
    for (; c < ce; ++c) {
        if (!cross) {
            sp.at = c * CH;
            sp.seg = (int)ring_segment(sp.at, ly.n, od.ng);
            sp.hi = segment_end(sp.seg, ly.n, od.ng);
            if (sp.hi < min(sp.at + CH, ly.n)) continue;  // crosses: one of the first blocks, or of a launch of its own
        }
        ex_chunk<V, HW, KAHAN, CROSS && ONE ? EX_BOTH : EX_WHOLE>(a, ly, pal, od, c, sp, cur, pd);
    }
    flush_out(a, pd);
}

// One element through the whole ordered chain, any variant.
template <int V, bool KAHAN>
__device__ float reduce_elem_ex(const ReduceArgs& a, const FmtK& f, int64_t j, int F, int seg, const Order& od) {
    bool bad = false;
    const int k = 1 << od.log2k;
    auto q = [&](int r) { return quant<V>(a.G[(int64_t)order_row(r, seg, od) * a.ld + j], F, f, bad); };
    float T = 0.0f, cT = 0.0f;
    for (int gi = 0; gi < od.ng; ++gi) {
        float S = q(gi * k), cS = 0.0f;
        for (int m = 1; m < k; ++m) chain_step<V, KAHAN>(S, cS, q(gi * k + m), f, bad);
        if (gi == 0)
            T = S;
        else
            chain_step<V, KAHAN>(T, cT, S, f, bad);
    }
    return finish<V>(T, bad);
}

template <bool KAHAN>
__device__ float reduce_elem_ex_any(const ReduceArgs& a, const FmtK& f, int64_t j, int F, int seg, const Order& od) {
    switch (f.variant) {
        case V_INT_F32: return reduce_elem_ex<V_INT_F32, KAHAN>(a, f, j, F, seg, od);
        case V_INT_F64: return reduce_elem_ex<V_INT_F64, KAHAN>(a, f, j, F, seg, od);
        case V_INT_EXACT: return reduce_elem_ex<V_INT_EXACT, KAHAN>(a, f, j, F, seg, od);
        case V_INT_M0: return reduce_elem_ex<V_INT_M0, KAHAN>(a, f, j, F, seg, od);
        case V_TOP_F32: return reduce_elem_ex<V_TOP_F32, KAHAN>(a, f, j, F, seg, od);
        case V_TOP_F64: return reduce_elem_ex<V_TOP_F64, KAHAN>(a, f, j, F, seg, od);
        case V_TOP_M0: return reduce_elem_ex<V_TOP_M0, KAHAN>(a, f, j, F, seg, od);
        case V_LOW_F32: return reduce_elem_ex<V_LOW_F32, KAHAN>(a, f, j, F, seg, od);
        case V_LOW_F64: return reduce_elem_ex<V_LOW_F64, KAHAN>(a, f, j, F, seg, od);
        case V_GEN: return reduce_elem_ex<V_GEN, KAHAN>(a, f, j, F, seg, od);
        default: return reduce_elem_ex<V_LOW_M0, KAHAN>(a, f, j, F, seg, od);
    }
}

// Chunks that mix palette entries, one block per chunk (blocks of other
// chunks return at once); element pairs per thread so that a byte of nibble
// codes has one writer.
template <bool KAHAN>
__global__ __launch_bounds__(BLOCK) void k_sim_reduce_ex_slow(ReduceArgs a, Layers ly, Pal pal, Order od) {
    __shared__ FmtK spal[APS_MAX_FORMATS];
    pal_to_lds(pal, spal);
    const int64_t start = (int64_t)blockIdx.x * CH;
    if (start >= ly.n) return;
    const int64_t end = min(start + CH, ly.n);
    const ChunkInfo ci = chunk_layers(ly, start, end);
    if (!ci.mixed) return;
    for (int64_t j0 = start + 2 * (int64_t)threadIdx.x; j0 < end; j0 += 2 * BLOCK) {
        uint32_t cd[2] = {0, 0};
        for (int e = 0; e < 2; ++e) {
            const int64_t j = j0 + e;
            if (j >= end) break;
            const int li = find_layer(ly.offsets, ly.L, j, 0);
            const FmtK& f = spal[ly.fmt_idx ? ly.fmt_idx[li] : 0];
            const int32_t ft = ly.scale_exp ? clamp_exp(ly.scale_exp[li]) : 0;
            const int F = ((a.flags & APS_INPUT_QUANTIZED) ? 0 : ft) + f.k;
            const int Fo = -(((a.flags & APS_OUTPUT_SCALED) ? 0 : ft) + f.k);
            const float sv = reduce_elem_ex_any<KAHAN>(a, f, j, F, (int)ring_segment(j, ly.n, od.ng), od);
            if (a.out) a.out[j] = __builtin_amdgcn_ldexpf(sv, Fo);
            cd[e] = encode(__builtin_amdgcn_ldexpf(sv, -f.k), f);
            if (a.codes && a.code_cls != 0) put_code(a.codes, j, cd[e], a.code_cls);
        }
        if (a.codes && a.code_cls == 0) {
            uint8_t* q = a.codes + (j0 >> 1);
            *q = (j0 + 1 < end) ? (uint8_t)((cd[0] & 15u) | ((cd[1] & 15u) << 4))
                                : (uint8_t)((*q & 0xF0u) | (cd[0] & 15u));
        }
    }
}

}  // namespace aps

using namespace aps;

extern "C" int aps_sim_reduce_ex(const float* G, int32_t W, int64_t ld, int64_t n, const int64_t* offsets,
                                 int32_t L, const int32_t* scale_exp, const aps_format* fmts, int32_t n_fmts,
                                 const uint8_t* fmt_idx, uint32_t flags, const aps_reduce_opts* opts, float* out,
                                 void* codes_out, void* stream) {
    const int32_t group = opts ? opts->group : W;
    const int32_t acc = opts ? opts->accumulator : APS_ACC_SEQUENTIAL;
    if (acc != APS_ACC_SEQUENTIAL && acc != APS_ACC_KAHAN) return APS_ERR_UNSUPPORTED;
    if (group < 1 || (group & (group - 1)) != 0 || W % group != 0) {
        // validate the rest first so that the size error is not masked
        const int st = check_rows(G, W, ld, n, offsets, L);
        return st != APS_OK ? st : APS_ERR_SIZE;
    }
    if (group == W && acc == APS_ACC_SEQUENTIAL)
        return aps_sim_reduce(G, W, ld, n, offsets, L, scale_exp, fmts, n_fmts, fmt_idx, flags, out, codes_out,
                              stream);
    int st = check_rows(G, W, ld, n, offsets, L);
    if (st != APS_OK) return st;
    if (!out && !codes_out && n > 0) return APS_ERR_NULL;
    if ((out && !aligned16(out)) || (codes_out && !aligned16(codes_out))) return APS_ERR_ALIGN;
    if (flags & ~(APS_INPUT_QUANTIZED | APS_OUTPUT_SCALED)) return APS_ERR_UNSUPPORTED;
    Pal pal;
    int ccls = 0;
    st = check_palette(fmts, n_fmts, pal, &ccls);
    if (st != APS_OK) return st;
    if (codes_out && (ccls < 0 || ccls > 2)) return APS_ERR_UNSUPPORTED;
    if (n == 0) return APS_OK;
    hipStream_t s = (hipStream_t)stream;
    Layers ly{offsets, fmt_idx, scale_exp, n, L, n_fmts};
    ReduceArgs a{G, out, (uint8_t*)codes_out, ld, W, flags, ccls, nullptr, nullptr};
    Order od{__builtin_ctz((unsigned)group), W / group};
    const int64_t nchunks = (n + CH - 1) / CH;
    one_form_per_variant(
        pal, n_fmts, [](const FmtK& f) { return f.variant; }, [](const FmtK& f) { return hw_of_chain(f); });
    unsigned vm = 0, hm = 0;  // variants of the entries without, and forms of those with, hardware chains
    for (int i = 0; i < n_fmts; ++i) {
        const int hw = hw_of_chain(pal.f[i]);
        if (hw) hm |= 1u << hw;
        else vm |= 1u << pal.f[i].variant;
    }
    // as many blocks as chunks can cross ring segments (the number of
    // boundaries alone would take the grid past its limit of 2^32 threads at
    // W = 2^24)
    const int ncross = (int)std::min<int64_t>(od.ng - 1, nchunks);
    const dim3 grid((unsigned)(grid_for(nchunks, BLOCKS_PER_CU) + ncross));
#define APS_XL(v, h, kahan, cross) \
    hipLaunchKernelGGL((k_sim_reduce_ex<v, h, kahan, cross>), grid, dim3(BLOCK), 0, s, a, ly, pal, od, ncross)
#define APS_X(v, h)                                                      \
    if (acc == APS_ACC_KAHAN) {                                          \
        if (ncross) APS_XL(v, h, true, true); else APS_XL(v, h, true, false);   \
    } else {                                                             \
        if (ncross) APS_XL(v, h, false, true); else APS_XL(v, h, false, false); \
    }
    if (hm & (1u << HW_E5M2)) { APS_X(V_TOP_F32, HW_E5M2) }
    if (hm & (1u << HW_HALF)) { APS_X(V_TOP_F32, HW_HALF) }
#define APS_LAUNCH_X(v) \
    if (vm & (1u << (v))) { APS_X(v, HW_NONE) }
    APS_FOR_VARIANTS(APS_LAUNCH_X)
#undef APS_LAUNCH_X
#undef APS_X
#undef APS_XL
    if (fmt_idx && n_fmts > 1 && L > 1) {  // chunks that mix palette entries
        if (acc == APS_ACC_KAHAN)
            hipLaunchKernelGGL(k_sim_reduce_ex_slow<true>, dim3((unsigned)nchunks), dim3(BLOCK), 0, s, a, ly, pal, od);
        else
            hipLaunchKernelGGL(k_sim_reduce_ex_slow<false>, dim3((unsigned)nchunks), dim3(BLOCK), 0, s, a, ly, pal, od);
    }
    return launched();
}
