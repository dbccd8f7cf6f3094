// One verification layer around the trajectory-masked attention (a pre-norm decoder layer of
// the 8B-shaped diffusion LMs the method runs on): the elementwise kernels between the
// library GEMMs (SwiGLU belongs to the gate / up projection).  All activations are bf16 in HBM,
// arithmetic in fp32.
//   rmsnorm_kernel     out = x / sqrt(mean(x^2) + eps) * w            (one workgroup per token); after a
//                      split projection it also adds the partial products to the residual stream
//   rope_split_kernel  [q | k | v] rows of the QKV projection -> q, k_draft, v_draft in the
//                      attention's layouts, rotary position embedding on q and k (pairs d and
//                      d + D/2, angle = pos * theta^(-2d/D)); token p of every draft of a block
//                      sits at position pos0[b] + p (the drafts are alternative states of the
//                      same block).  In the dual-cache refresh it also writes the rotated K / V rows outside the
//                      current block into the prefix | suffix cache
#pragma once

#include "common.hpp"
#include "gemm.hpp"

namespace trajspec {

constexpr int kLayerThreads = 256;
constexpr int kLayerMaxHalf = 64;  // D / 2 for the head sizes the attention supports (64, 128)

__device__ __forceinline__ uint16_t f2bf(float f) {
    return __builtin_bit_cast(uint16_t, (__bf16)f);  // round to nearest even
}

// Sum over a workgroup of THREADS threads, in every thread.
template <int THREADS>
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) t += red[w];
    return t;
}

__device__ __forceinline__ float square_sum8(const u32x4_t& v) {
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = bf16_lo(v[e]), b = bf16_hi(v[e]);
        ss += a * a + b * b;
    }
    return ss;
}

__device__ __forceinline__ u32x4_t norm8(const u32x4_t& v, float inv, const u32x4_t& g) {
    u32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = bf16_lo(v[e]) * inv * bf16_lo(g[e]);
        const float b = bf16_hi(v[e]) * inv * bf16_hi(g[e]);
        o[e] = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
    }
    return o;
}

// x, out: [T, hidden] bf16 (rows contiguous); w: [hidden].  hidden % 8 == 0, R = chunks of 8 per
// thread, or 0 for rows of any length.  With SPLIT the row first becomes x + the sum of the `splits`
// partial products [T, hidden] of the projection before it (rounded once, written back to x).
// A few rows' norm is a chain of memory latencies: the row, the weights and the partial products are
// all requested before anything waits and the row stays in registers (64 x 4096 rows: 4.8 -> 3 us
// with the weights' cold miss behind the row's, and one launch instead of two after a split).
template <int THREADS, int R, bool SPLIT>
__global__ __launch_bounds__(THREADS) void rmsnorm_kernel(uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
                                                          uint16_t* __restrict__ out, int hidden, float eps,
                                                          const float* __restrict__ partial, int splits) {
    __shared__ float red[THREADS / 64];
    uint16_t* xr = x + (int64_t)blockIdx.x * hidden;
    uint16_t* orow = out + (int64_t)blockIdx.x * hidden;
    const int nv = hidden / 8;
    const int64_t TN = (int64_t)gridDim.x * hidden;
    float ss = 0.f;
    if (R > 0) {
        u32x4_t v[R > 0 ? R : 1], g[R > 0 ? R : 1];
        float p[R > 0 ? R : 1][8];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * THREADS;
            const int at = i < nv ? i : 0;
            v[r] = *reinterpret_cast<const u32x4_t*>(xr + 8 * at);
            g[r] = *reinterpret_cast<const u32x4_t*>(w + 8 * at);
            if (SPLIT) split_sum8(partial, splits, TN, (int64_t)blockIdx.x * hidden + 8 * at, p[r]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * THREADS;
            if (SPLIT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    p[r][2 * e] += bf16_lo(v[r][e]);
                    p[r][2 * e + 1] += bf16_hi(v[r][e]);
                }
                v[r] = round8(p[r]);
                if (i < nv) *reinterpret_cast<u32x4_t*>(xr + 8 * i) = v[r];
            }
            if (i < nv) ss += square_sum8(v[r]);
        }
        const float inv = 1.0f / sqrtf(block_sum<THREADS>(ss, red) / (float)hidden + eps);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = threadIdx.x + r * THREADS;
            if (i < nv) *reinterpret_cast<u32x4_t*>(orow + 8 * i) = norm8(v[r], inv, g[r]);
        }
        return;
    }
    for (int i = threadIdx.x; i < nv; i += THREADS) {
        u32x4_t v = *reinterpret_cast<const u32x4_t*>(xr + 8 * i);
        if (SPLIT) {
            float p[8];
            split_sum8(partial, splits, TN, (int64_t)blockIdx.x * hidden + 8 * i, p);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[2 * e] += bf16_lo(v[e]);
                p[2 * e + 1] += bf16_hi(v[e]);
            }
            v = round8(p);
            *reinterpret_cast<u32x4_t*>(xr + 8 * i) = v;  // read back by the same thread below
        }
        ss += square_sum8(v);
    }
    const float inv = 1.0f / sqrtf(block_sum<THREADS>(ss, red) / (float)hidden + eps);
    for (int i = threadIdx.x; i < nv; i += THREADS)
        *reinterpret_cast<u32x4_t*>(orow + 8 * i) =
            norm8(*reinterpret_cast<const u32x4_t*>(xr + 8 * i), inv, *reinterpret_cast<const u32x4_t*>(w + 8 * i));
}

// qkv: [T, (Hq + 2 Hkv) D] rows [q heads | k heads | v heads]; token t = (b N + n) L + p.
// q: [T, Hq, D], kd / vd: [T, Hkv, D].  One workgroup (few tokens: several, grid y) per token: the
// D / 2 rotation angles depend on the position only, so they are computed once per workgroup (into LDS);
// every head then moves 16-byte chunks (8 elements of the first half and the matching 8 of the
// second).  D % 16 == 0.  With SPLIT the rows are the sums of the projection's `splits` partial
// products, rounded to bf16.  A thread's first two pairs of chunks are requested before the angles are computed.
// CacheRows: where the refresh also puts the K and V rows of the positions outside each sequence's block
// [block_start[b], block_start[b] + L): [B, S, Hkv D], prefix rows then suffix rows (a block_start
// outside [0, S] is reported and clamped).  kc == null: nowhere.
struct CacheRows {
    const int32_t* block_start;
    uint16_t *kc, *vc;
    int S, L;
};

template <bool SPLIT>
__global__ __launch_bounds__(kLayerThreads) void rope_split_kernel(const uint16_t* __restrict__ qkv,
                                                                   const float* __restrict__ partial, int splits,
                                                                   const int32_t* __restrict__ pos0,
                                                                   uint16_t* __restrict__ q, uint16_t* __restrict__ kd,
                                                                   uint16_t* __restrict__ vd, int NL, int L, int Hq,
                                                                   int Hkv, int D, float log2_theta, CacheRows cache) {
    __shared__ float cs[kLayerMaxHalf], sn[kLayerMaxHalf];
    const int t = blockIdx.x;
    const int b = t / NL;
    const int p = t % L;
    const int half = D / 2;
    const int width = (Hq + 2 * Hkv) * D;
    const int64_t row = (int64_t)t * width, TW = (int64_t)gridDim.x * width;
    auto chunk = [&](int at) -> u32x4_t {
        if (SPLIT) {
            float v[8];
            split_sum8(partial, splits, TW, row + at, v);
            return round8(v);
        }
        return *reinterpret_cast<const u32x4_t*>(qkv + row + at);
    };
    // tasks: rotated pairs of chunks of the q and k heads (head, chunk of 8 in the first half), then
    // pairs of chunks of the v heads (copied)
    const int cpr = half / 8;  // chunks per half
    const int rotated = (Hq + Hkv) * cpr, tasks = rotated + Hkv * cpr;
    auto load = [&](int i, u32x4_t& a, u32x4_t& c) {
        const int head = i / cpr, at = head * D + 8 * (i - head * cpr);  // v heads follow the k heads
        a = chunk(at);
        c = chunk(at + half);
    };
    const int pos = pos0 != nullptr ? pos0[b] + p : p;
    u32x4_t a0, c0, a1 = {}, c1 = {};
    const int first = blockIdx.y * kLayerThreads + threadIdx.x, stride = gridDim.y * kLayerThreads;
    const int i0 = first, i1 = first + stride;
    load(i0 < tasks ? i0 : 0, a0, c0);
    if (stride < tasks) load(i1 < tasks ? i1 : 0, a1, c1);  // uniform: a few tokens' threads have one pair
    for (int d = threadIdx.x; d < half; d += kLayerThreads) {
        const float inv_freq = exp2f(-(2.0f * d / (float)D) * log2_theta);
        sincosf((float)pos * inv_freq, &sn[d], &cs[d]);
    }
    int64_t cache_row = -1;  // of this token, or none
    if (cache.kc != nullptr) {
        int bs = cache.block_start[b];
        if (bs < 0 || bs > cache.S) {
            if (p == 0 && blockIdx.y == 0 && threadIdx.x == 0) flag_device_status(4);
            bs = bs < 0 ? 0 : cache.S;
        }
        if (p < bs || p >= bs + cache.L) cache_row = (int64_t)b * cache.S + (p < bs ? p : p - cache.L);
    }
    __syncthreads();
    auto finish = [&](int i, const u32x4_t& a, const u32x4_t& c) {
        const int head = i / cpr, d0 = 8 * (i - head * cpr);
        u32x4_t lo = a, hi = c;
        if (i < rotated) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int d = d0 + 2 * e;
                const float x1a = bf16_lo(a[e]), x1b = bf16_hi(a[e]);
                const float x2a = bf16_lo(c[e]), x2b = bf16_hi(c[e]);
                lo[e] = (uint32_t)f2bf(x1a * cs[d] - x2a * sn[d]) | ((uint32_t)f2bf(x1b * cs[d + 1] - x2b * sn[d + 1]) << 16);
                hi[e] = (uint32_t)f2bf(x2a * cs[d] + x1a * sn[d]) | ((uint32_t)f2bf(x2b * cs[d + 1] + x1b * sn[d + 1]) << 16);
            }
        }
        uint16_t* dst = head < Hq         ? q + ((int64_t)t * Hq + head) * D
                        : head < Hq + Hkv ? kd + ((int64_t)t * Hkv + (head - Hq)) * D
                                          : vd + ((int64_t)t * Hkv + (head - Hq - Hkv)) * D;
        *reinterpret_cast<u32x4_t*>(dst + d0) = lo;
        *reinterpret_cast<u32x4_t*>(dst + d0 + half) = hi;
        if (cache_row >= 0 && head >= Hq) {
            const int kv = head - Hq;  // k heads, then v heads
            uint16_t* c = (kv < Hkv ? cache.kc : cache.vc) + (cache_row * Hkv + (kv < Hkv ? kv : kv - Hkv)) * D;
            *reinterpret_cast<u32x4_t*>(c + d0) = lo;
            *reinterpret_cast<u32x4_t*>(c + d0 + half) = hi;
        }
    };
    if (i0 < tasks) finish(i0, a0, c0);
    if (i1 < tasks) finish(i1, a1, c1);
    for (int i = first + 2 * stride; i < tasks; i += stride) {
        load(i, a0, c0);
        finish(i, a0, c0);
    }
}

}  // namespace trajspec
