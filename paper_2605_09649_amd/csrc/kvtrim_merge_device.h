// Merging of a segment's partial attention results by the last of its blocks to finish, used where a launch of the merge
// kernel would cost more than the blocks' meeting.
#pragma once
#include "kvtrim_device.h"

namespace kvtrim {

// The first query head (row of q, out and lse) of segment seg.
template <int G>
__device__ __forceinline__ int64_t q_row_of(int seg, const Shape& sh) {
    const int seq = seg / sh.segs_per_seq, lh = seg - seq * sh.segs_per_seq;
    const int layer = lh / sh.n_kv_heads, head = lh - layer * sh.n_kv_heads;
    return ((int64_t)seq * sh.n_layers + layer) * sh.n_q_heads + (int64_t)head * G;
}

// Stores past the caches that are not coherent across the chip: once acknowledged, another block reads them by merge_shared.
__device__ __forceinline__ void put_shared(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Maximum and sum over the wavefront, in every lane: by DPP inside the rows of 16 lanes and then across them, without LDS.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_or(float v, float other) {   // `other` where there is no such lane
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(other), __float_as_int(v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp_or<0x111, 0xF>(v, -INFINITY));
    v = fmaxf(v, dpp_or<0x112, 0xF>(v, -INFINITY));
    v = fmaxf(v, dpp_or<0x114, 0xF>(v, -INFINITY));
    v = fmaxf(v, dpp_or<0x118, 0xF>(v, -INFINITY));
    v = fmaxf(v, dpp_or<0x142, 0xA>(v, -INFINITY));
    v = fmaxf(v, dpp_or<0x143, 0xC>(v, -INFINITY));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_total(float v) {
    v += dpp_or<0x111, 0xF>(v, 0.f);
    v += dpp_or<0x112, 0xF>(v, 0.f);
    v += dpp_or<0x114, 0xF>(v, 0.f);
    v += dpp_or<0x118, 0xF>(v, 0.f);
    v += dpp_or<0x142, 0xA>(v, 0.f);
    v += dpp_or<0x143, 0xC>(v, 0.f);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// The last block of a segment to finish merges: the n partial results at `part` ([n][G][D + 2] = (m in base-2 units, l,
// o[D] unnormalised)) become the segment's output.  A thread owns two columns of a head and every
// RG-th partial result; their loads and those of the (m, l) pairs, a lane per result, go out together, so a tile of results
// costs one round trip.  The results come past the caches that are not coherent across the chip (eight bytes a load).
template <int D, int G, int THREADS>
__device__ __forceinline__ void merge_shared(const float* __restrict__ part, int n, int64_t hq, float* lds, float* __restrict__ out,
                                             float* __restrict__ lse) {
    constexpr int PAIRS = G * D / 2;                              // 32 .. 512
    constexpr int RG = THREADS / PAIRS > 4 ? 4 : THREADS / PAIRS; // groups of threads that share the results
    constexpr int LOADS = 16, TILE = RG * LOADS;                  // 16 .. 64 results
    static_assert(RG >= 1 && TILE <= 64 && THREADS / 64 >= G, "a wavefront for every head, a lane for every result of a tile");
    float2* s_acc = reinterpret_cast<float2*>(lds);               // [RG - 1][PAIRS]
    float* s_w = lds + 2 * (RG - 1) * PAIRS;                      // [G][TILE] weights of a tile's results
    float* s_scale = s_w + G * TILE;                              // [G] what the sums so far are scaled by
    float* s_ml = s_scale + G;                                    // [G][2] maximum and denominator
    static_assert(2 * (RG - 1) * PAIRS + G * TILE + 3 * G <= THREADS / 64 * G * (D + 8), "fits the wavefronts' partial results");
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = tid / PAIRS, pair = tid - rg * PAIRS, g = pair / (D / 2), col = 2 * (pair - g * (D / 2));
    const bool mine = rg < RG;
    auto ld2 = [](const float* p) {
        return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    constexpr size_t stride = (size_t)G * (D + 2);
    float2 acc = make_float2(0.f, 0.f);
    float M = -INFINITY, L = 0.f;                                 // of head `wave`
    for (int t0 = 0; t0 < n; t0 += TILE) {
        float2 x[LOADS];
        float2 ml = make_float2(-INFINITY, 0.f);
        if (wave < G && lane < TILE && t0 + lane < n) ml = ld2(part + (t0 + lane) * stride + (size_t)wave * (D + 2));
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int e = t0 + u * RG + rg;
            x[u] = make_float2(0.f, 0.f);
            if (mine && e < n) x[u] = ld2(part + e * stride + (size_t)g * (D + 2) + 2 + col);
        }
        if (wave < G) {
            const float Mn = fmaxf(M, wave_max(ml.x)), ms = Mn == -INFINITY ? 0.f : Mn;
            const float alpha = __builtin_amdgcn_exp2f(M - ms), w = __builtin_amdgcn_exp2f(ml.x - ms);   // (2^-inf = 0)
            L = L * alpha + wave_total(ml.y * w);
            M = Mn;
            if (lane < TILE) s_w[wave * TILE + lane] = w;
            if (lane == 0) {
                s_scale[wave] = alpha;
                s_ml[2 * wave] = M;
                s_ml[2 * wave + 1] = L;
            }
        }
        __syncthreads();
        if (mine) {
            const float a = s_scale[g];
            acc.x *= a;
            acc.y *= a;
#pragma unroll
            for (int u = 0; u < LOADS; ++u) {
                const float w = s_w[g * TILE + u * RG + rg];
                acc.x = fmaf(x[u].x, w, acc.x);
                acc.y = fmaf(x[u].y, w, acc.y);
            }
        }
        __syncthreads();
    }
    if (RG > 1) {
        if (mine && rg > 0) s_acc[(rg - 1) * PAIRS + pair] = acc;
        __syncthreads();
        if (rg == 0) {
#pragma unroll
            for (int k = 0; k < RG - 1; ++k) {
                const float2 o = s_acc[k * PAIRS + pair];
                acc.x += o.x;
                acc.y += o.y;
            }
        }
    }
    if (rg == 0) {
        const float l = s_ml[2 * g + 1];
        float* o = out + (hq + g) * D + col;                      // (one by one: the caller's array need not be 8-byte aligned)
        o[0] = l > 0.f ? acc.x / l : 0.f;
        o[1] = l > 0.f ? acc.y / l : 0.f;
        if (col == 0 && lse) lse[hq + g] = l > 0.f ? (s_ml[2 * g] + __builtin_amdgcn_logf(l)) * 0.6931471805599453f : -INFINITY;
    }
    __syncthreads();                                              // (LDS may be used again)
}

}  // namespace kvtrim
