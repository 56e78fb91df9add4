// aps_small.hip -- one whole APS synchronisation (Algorithm 1 with the
// low-precision accumulator of Sec. 5) of a small set in two launches.
#include "aps_common.hpp"

namespace aps {

// ======================================================= K5c: small sets
//
// A set that stays in the caches takes a few microseconds per launch whatever
// it computes: the launch itself (about 4 us of the host's time), the first
// read of the kernel's arguments, one trip to memory after another.  So here
// the step is two launches that pass one value between them: the first
// writes every unit's maximum per layer, the second reads a layer's maxima
// back, derives the exponent and sums through the scaled path, with its rows
// already on their way while it does.  Nothing is accumulated, so nothing has
// to be cleared first.
//
// A unit is the 256 elements of one wave (4 per lane).  Walking the units and
// the layers in order, the pair (unit u, layer i) is new in u or in i, so
// u + i numbers the pairs, and a layer's maxima are consecutive: for layer i
// of units u0..u1, entries u0 + i .. u1 + i.

constexpr int64_t UNIT = 64 * VEC;

// Where the layers start inside a wave's unit: each of a lane's 4 elements
// gets the position, within the unit, of its layer's first element there.
// The first layers' positions are scattered to LDS, and a running maximum
// over the positions carries each to the elements after it.
__device__ __forceinline__ void layer_starts(const Layers& ly, const ChunkInfo& ci, int64_t start, int64_t end,
                                             uint32_t* mark, uint32_t pos[4]) {
    const int lane = threadIdx.x & 63;
    *(u4v*)(mark + 4 * lane) = u4v{0u, 0u, 0u, 0u};
    wave_lds_sync();
    for (int64_t i = ci.i0 + lane; i <= ci.i1; i += 64) {
        const int64_t lo = ly.offsets[i];
        if (lo > start && lo < end && ly.offsets[i + 1] > lo) mark[lo - start] = (uint32_t)(lo - start);
    }
    wave_lds_sync();
    const u4v m = *(const u4v*)(mark + 4 * lane);
    pos[0] = m.x;
    pos[1] = max(m.y, pos[0]);
    pos[2] = max(m.z, pos[1]);
    pos[3] = max(m.w, pos[2]);
    uint32_t before = pos[3];  // maximum over the lanes up to this one
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = (uint32_t)__shfl_up((int)before, o, 64);
        if (lane >= o) before = max(before, up);
    }
    const uint32_t prev = (uint32_t)__shfl_up((int)before, 1, 64);
    if (lane > 0)
        for (int e = 0; e < 4; ++e) pos[e] = max(pos[e], prev);
    wave_lds_sync();
}

// Every unit's maximum magnitude per layer.
__global__ __launch_bounds__(BLOCK) void k_small_max(const float* __restrict__ G, int32_t W, int64_t ld, Layers ly,
                                                    uint32_t* __restrict__ part) {
    __shared__ __align__(16) uint32_t smark[BLOCK / 64][UNIT], smax[BLOCK / 64][UNIT];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t u = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (BLOCK / 64) + wv));
    const int64_t start = u * UNIT;
    if (start >= ly.n) return;
    const int64_t end = min(start + UNIT, ly.n);
    const int64_t j = start + lane * VEC;
    uint32_t m[4] = {0u, 0u, 0u, 0u};
    if (j < end) {
        const float* p = G + j;
        // batches of MAXABS_UNROLL rows; rows past W-1 re-read row W-1
        for (int w = 0; w < W; w += MAXABS_UNROLL) {
            f4 x[MAXABS_UNROLL];
#pragma unroll
            for (int r = 0; r < MAXABS_UNROLL; ++r) x[r] = *(const f4*)(p + (int64_t)min(w + r, W - 1) * ld);
#pragma unroll
            for (int r = 0; r < MAXABS_UNROLL; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = max(m[e], f2u(x[r][e]) & 0x7FFFFFFFu);
        }
        for (int e = 1; e < 4; ++e)
            if (j + e >= end) m[e] = 0;  // row padding does not count
    }
    const ChunkInfo ci = chunk_layers(ly, start, end);
    if (ci.i0 == ci.i1) {
        const uint32_t v = wave_max_u32(max(max(m[0], m[1]), max(m[2], m[3])));
        if (lane == 0) part[u + ci.i0] = v;
        return;
    }
    uint32_t pos[4];
    layer_starts(ly, ci, start, end, smark[wv], pos);
    *(u4v*)(smax[wv] + 4 * lane) = u4v{0u, 0u, 0u, 0u};
    wave_lds_sync();
    for (int e = 0; e < 4; ++e)
        if (m[e]) atomicMax(&smax[wv][pos[e]], m[e]);
    wave_lds_sync();
    for (int64_t i = ci.i0 + lane; i <= ci.i1; i += 64) {
        const int64_t lo = max(ly.offsets[i], start), hi = min(ly.offsets[i + 1], end);
        if (lo < hi) part[u + i] = smax[wv][lo - start];
    }
}

// The maximum over a layer's units, by the whole wave.
__device__ __forceinline__ uint32_t layer_max(const Layers& ly, const uint32_t* __restrict__ part, int i) {
    const int64_t u0 = cld(ly.offsets, i) / UNIT, u1 = (cld(ly.offsets, i + 1) - 1) / UNIT;
    uint32_t v = 0;
    for (int64_t k = u0 + (threadIdx.x & 63); k <= u1; k += 64) v = max(v, part[k + i]);
    return wave_max_u32(v);
}

template <int V>
__global__ __launch_bounds__(BLOCK) void k_small_sum(ReduceArgs a, Layers ly, FmtK f,
                                                    const uint32_t* __restrict__ part, uint32_t* __restrict__ maxabs,
                                                    int32_t* __restrict__ scale_exp) {
    __shared__ __align__(16) uint32_t smark[BLOCK / 64][UNIT];
    __shared__ int32_t sft[BLOCK / 64][UNIT];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // empty layers belong to no unit
    for (int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x; i < ly.L; i += (int64_t)gridDim.x * BLOCK)
        if (ly.offsets[i] == ly.offsets[i + 1]) {
            maxabs[i] = 0u;
            scale_exp[i] = 0;
        }
    const int64_t u = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * (BLOCK / 64) + wv));
    const int64_t start = u * UNIT;
    if (start >= ly.n) return;
    const int64_t end = min(start + UNIT, ly.n);
    const int64_t j = start + lane * VEC;
    const float* p = a.G + (j < end ? j : start);  // a lane past the end sums the unit's start and stores nothing
    const int64_t ld = a.ld;
    const f4 neg0 = {-0.0f, -0.0f, -0.0f, -0.0f};
    int F[4];
    float s[4];
    bool bad[4] = {false, false, false, false};
    stream_rows(
        a.W, [&](int r) { return *(const f4*)(p + (int64_t)r * ld); },
        [&]() {  // the exponents, with the first rows' loads in flight
            const ChunkInfo ci = chunk_layers(ly, start, end);
            // the wave of a layer's first unit writes its maximum and exponent
            auto one = [&](int i) {
                const uint32_t mx = layer_max(ly, part, i);
                const int32_t r = scale_of(mx, a.W, f.emax);
                if (lane == 0 && cld(ly.offsets, i) >= start) {
                    maxabs[i] = mx;
                    scale_exp[i] = r;
                }
                return r;
            };
            const int32_t first = one(ci.i0);
            int32_t ft[4] = {first, first, first, first};
            if (ci.i0 != ci.i1) {
                // a layer between the first and the last lies inside the unit
                const bool more = ci.i1 > ci.i0 && cld(ly.offsets, ci.i1) < cld(ly.offsets, ci.i1 + 1);
                const int32_t last = more ? one(ci.i1) : first;
                uint32_t pos[4];
                layer_starts(ly, ci, start, end, smark[wv], pos);
                for (int64_t i = ci.i0 + lane; i <= ci.i1; i += 64) {
                    const int64_t lo = max(ly.offsets[i], start), hi = min(ly.offsets[i + 1], end);
                    if (lo >= hi) continue;
                    int32_t r = i == ci.i0 ? first : last;
                    if (i != ci.i0 && i != ci.i1) {
                        const uint32_t mx = part[u + i];
                        r = scale_of(mx, a.W, f.emax);
                        maxabs[i] = mx;
                        scale_exp[i] = r;
                    }
                    sft[wv][lo - start] = r;
                }
                wave_lds_sync();
                for (int e = 0; e < 4; ++e) ft[e] = sft[wv][pos[e]];
            }
            for (int e = 0; e < 4; ++e) F[e] = clamp_exp(ft[e]) + f.k;
        },
        [&](const f4& x) {
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = quant<V>(x[e], F[e], f, bad[e]);
        },
        [&](const f4& r, bool valid) {
            const f4 v = valid ? r : neg0;
#pragma unroll
            for (int e = 0; e < 4; ++e) s[e] = accum<V>(s[e], quant<V>(v[e], F[e], f, bad[e]), f, bad[e]);
        });
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = __builtin_amdgcn_ldexpf(finish<V>(s[e], bad[e]), -F[e]);
    if (j + 4 <= end) {
        *(f4*)(a.out + j) = o;
    } else {
        for (int e = 0; e < 4 && j + e < end; ++e) a.out[j + e] = o[e];
    }
}

void launch_sync_small(const ReduceArgs& a, const Layers& ly, const FmtK& f, uint32_t* part, uint32_t* maxabs,
                       int32_t* scale_exp, hipStream_t s) {
    const int64_t units = (ly.n + UNIT - 1) / UNIT;
    const int64_t blocks = (units + BLOCK / 64 - 1) / (BLOCK / 64);
    if (ly.n > 0) hipLaunchKernelGGL(k_small_max, dim3((unsigned)blocks), dim3(BLOCK), 0, s, a.G, a.W, a.ld, ly, part);
    const dim3 grid((unsigned)std::max<int64_t>(blocks, std::min<int64_t>((ly.L + BLOCK - 1) / BLOCK, 1024)));
#define APS_SM(v) \
    if (f.variant == (v)) hipLaunchKernelGGL(k_small_sum<v>, grid, dim3(BLOCK), 0, s, a, ly, f, part, maxabs, scale_exp);
    APS_FOR_VARIANTS(APS_SM)
#undef APS_SM
}

}  // namespace aps
