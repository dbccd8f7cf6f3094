// libtrajspec: C ABI of the gfx950 trajectory-verification step (see include/traj_spec.h).
// One translation unit: the kernels live in the headers included below.
#include <hip/hip_runtime.h>

#include <cmath>
#include <algorithm>
#include <climits>
#include <cstdint>
#include <mutex>

#include "../../include/traj_spec.h"
#include "accept.hpp"
#include "common.hpp"
#include "conf_topk.hpp"
#include "gemm.hpp"
#include "interblock.hpp"
#include "layer.hpp"
#include "tree.hpp"
#include "verify_attn.hpp"
#include "verify_attn16.hpp"

// Fixed device scratch of traj_confidence_topk_noalloc: the split records of short batches
// (at most TRAJ_TOPK_SCRATCH_BYTES).  Host code must not pass this name to a kernel or a copy: on
// the host it is only a handle; the device address comes from hipGetSymbolAddress, per device.
static __device__ __align__(256) unsigned char scratch[TRAJ_TOPK_SCRATCH_BYTES];

namespace {

using namespace trajspec;

// Device address of `scratch` on the current device, looked up once per device.
constexpr int kScratchMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kScratchMaxDevices];

traj_status device_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kScratchMaxDevices) return TRAJ_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return TRAJ_E_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return TRAJ_OK;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline traj_status launched() { return hipGetLastError() == hipSuccess ? TRAJ_OK : TRAJ_E_HIP; }

// ------------------------------------------------------------------ attention
traj_status check_attn(const traj_attn_shape* sh) {
    if (sh->B < 1 || sh->N < 1 || sh->L < 1 || sh->Hq < 1 || sh->Hkv < 1 || sh->S < 0) return TRAJ_E_SHAPE;
    if (sh->N > 64) return TRAJ_E_SHAPE;
    if (sh->Hq % sh->Hkv != 0) return TRAJ_E_SHAPE;
    if (sh->D != 64 && sh->D != 128) return TRAJ_E_UNSUPPORTED;
    if (!(sh->scale == sh->scale) || std::isinf(sh->scale)) return TRAJ_E_ARG;
    // flattened element counts must fit the kernels' 64-bit offsets and 32-bit row math
    const int64_t rows_per_group = (int64_t)(sh->Hq / sh->Hkv) * sh->N * sh->L;
    if (rows_per_group > (int64_t)1 << 30) return TRAJ_E_SHAPE;
    if ((int64_t)sh->S * sh->Hkv * sh->D > ((int64_t)1 << 40)) return TRAJ_E_SHAPE;
    // one sequence's cache slice is addressed through 32-bit buffer offsets
    if ((int64_t)sh->S * sh->Hkv * sh->D * 2 >= ((int64_t)1 << 31)) return TRAJ_E_UNSUPPORTED;
    return TRAJ_OK;
}

// Compute units of the current device (0 when the query fails).
int device_cu_count() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return cus;
}

// 16-row grids with a longer cache than this run two key groups per workgroup (two waves per SIMD,
// half the chain of steps each).  8 drafts x 32 heads x 128 dims, one group / two, cache from HBM and (near):
// 256 keys 11.0 / 11.4 us (10.8 / 11.2), 384 14.1 / 14.2 (12.0 / 12.5), 448 15.5 / 15.1 (12.8 / 12.9), 736 21.2 /
// 19.3 (16.7 / 15.9); up to 384 keys the merge costs what the steps save.
constexpr int kAttnSplitKeysMin = 384;
// The same for 32-row grids of at most one workgroup per CU, from this many keys on: 32 drafts x 32 heads over 512
// keys 19.4 / 20.2 us (20.0 / 21.1), 768 24.2 / 24.1 (25.2 / 26.0), 1024 28.7 / 27.5 (29.2 / 29.4), 1504 38.2 / 35.9
// (36.3 / 36.0); 16 drafts of 64 with 28 over 4 heads, 2048 keys 42.0 / 38.4 (39.6 / 38.9).
constexpr int kAttnSplitKeysMin32 = 1024;
// Weights per layer from which two layers displace a cache from the 256 MB last-level cache.
constexpr int64_t kAttnWarmLayerBytes = 128ll << 20;
// 16-row workgroups per kv head from which the cache is read ahead: each of them streams the whole head, and
// the read-ahead shares its first pass out between them.  Layers without / with it: 1 and 4 drafts of 32 heads (1
// and 2 workgroups), 736 keys 127.2 / 128.6 and 168.4 / 169.8 us, 5 drafts (3) 193.6 / 193.6, 7 drafts (4) 197.0 / 196.2,
// over 2048 keys 215.6 / 212.9; 32 over 8 heads, 2048 keys, 1 / 4 drafts (2 / 8) 135.5 / 136.7 and 180.2 / 172.8.
constexpr int kAttnWarmMinWorkgroups = 4;

// p describes the 32-row launch (4 waves x 32 rows per workgroup).  A grid that still has at
// most one workgroup per CU with 16-row waves (4 waves x 16 rows per workgroup, twice the
// workgroups) runs that way: each wave's chain of steps is half as long.  Larger grids keep
// 32-row waves: with two 16-row workgroups per CU the doubled LDS fragment reads and stage loads
// per MFMA cost more than the second wave per SIMD gains.
template <int D>
traj_status launch_attn(AttnParams p, hipStream_t st) {
    const int wg16 = (p.rows_per_group + kAttnWaves * 16 - 1) / (kAttnWaves * 16);
    const int64_t nwg16 = (int64_t)p.B * p.Hkv * wg16;
    if (nwg16 <= device_cu_count()) {
        p.wg_per_group = wg16;
        p.num_wg = (int)nwg16;
        if (wg16 < kAttnWarmMinWorkgroups) p.warm = 0;
        if (p.S > kAttnSplitKeysMin)
            hipLaunchKernelGGL((verify_attn16_kernel<D, 2>), dim3(p.num_wg), dim3(2 * kAttnThreads), 0, st, p);
        else
            hipLaunchKernelGGL((verify_attn16_kernel<D, 1>), dim3(p.num_wg), dim3(kAttnThreads), 0, st, p);
    } else {
        if (p.num_wg <= device_cu_count() && p.S >= kAttnSplitKeysMin32)
            hipLaunchKernelGGL((verify_attn_kernel<D, 2>), dim3(p.num_wg), dim3(2 * kAttnThreads), 0, st, p);
        else
            hipLaunchKernelGGL((verify_attn_kernel<D, 1>), dim3(p.num_wg), dim3(kAttnThreads), 0, st, p);
    }
    return launched();
}

traj_status verify_attn(const void* q, const void* k_cache, const void* v_cache, const void* k_draft, const void* v_draft,
                        const int32_t* draft_parent, const uint64_t* draft_peers, void* out, const traj_attn_shape* shape,
                        bool warm, hipStream_t s) {
    if (shape == nullptr || q == nullptr || k_draft == nullptr || v_draft == nullptr || draft_parent == nullptr ||
        out == nullptr)
        return TRAJ_E_NULL;
    if (shape->S > 0 && (k_cache == nullptr || v_cache == nullptr)) return TRAJ_E_NULL;
    traj_status st = check_attn(shape);
    if (st != TRAJ_OK) return st;
    if (!aligned16(q) || !aligned16(k_draft) || !aligned16(v_draft) || !aligned16(out) ||
        (shape->S > 0 && (!aligned16(k_cache) || !aligned16(v_cache))))
        return TRAJ_E_SHAPE;

    AttnParams p{};
    p.q = static_cast<const uint16_t*>(q);
    p.kc = static_cast<const uint16_t*>(k_cache);
    p.vc = static_cast<const uint16_t*>(v_cache);
    p.kd = static_cast<const uint16_t*>(k_draft);
    p.vd = static_cast<const uint16_t*>(v_draft);
    p.parent = draft_parent;
    p.peers = draft_peers;
    p.out = static_cast<uint16_t*>(out);
    p.B = shape->B;
    p.N = shape->N;
    p.L = shape->L;
    p.Hq = shape->Hq;
    p.Hkv = shape->Hkv;
    p.S = shape->S;
    p.group = shape->Hq / shape->Hkv;
    p.rows_per_group = p.group * p.N * p.L;
    const int rb = (p.rows_per_group + 31) / 32;
    p.wg_per_group = (rb + kAttnWaves - 1) / kAttnWaves;
    const int64_t nwg = (int64_t)p.B * p.Hkv * p.wg_per_group;
    if (nwg > 0x7fffffff) return TRAJ_E_SHAPE;
    p.num_wg = (int)nwg;
    const float scale = shape->scale > 0.f ? shape->scale : 1.0f / std::sqrt((float)shape->D);
    p.scale_log2 = scale * 1.4426950408889634f;
    p.drafts_visible = 1;
    p.warm = warm ? 1 : 0;
    return shape->D == 128 ? launch_attn<128>(p, s) : launch_attn<64>(p, s);
}

// ------------------------------------------------------------------ confidence / top-k
int vec_of(int32_t dtype) { return dtype == TRAJ_BF16 ? 8 : 4; }
int size_of(int32_t dtype) { return dtype == TRAJ_BF16 ? 2 : 4; }

traj_status check_logits(const traj_logits_shape* sh, int32_t k) {
    if (sh->dtype != TRAJ_BF16 && sh->dtype != TRAJ_F32) return TRAJ_E_DTYPE;
    if (sh->rows < 0 || sh->vocab < 1 || sh->vocab >= ((int64_t)1 << 31)) return TRAJ_E_SHAPE;
    if (sh->row_stride < sh->vocab) return TRAJ_E_SHAPE;
    if (sh->rows >= ((int64_t)1 << 31) / 64) return TRAJ_E_SHAPE;
    if (k < 1 || k > 8 || k > sh->vocab) return TRAJ_E_ARG;
    return TRAJ_OK;
}

template <typename T, int K, int THREADS, int U, int DEPTH>
void launch_conf_kernel(const T* lg, const traj_logits_shape* sh, int k, const TopkPlan& plan, float* conf,
                        int32_t* idx, float* partial, hipStream_t st) {
    const dim3 grid((unsigned)(sh->rows * plan.splits));
    hipLaunchKernelGGL((conf_topk_kernel<T, K, THREADS, U, DEPTH>), grid, dim3(THREADS), 0, st, lg,
                       sh->row_stride, (int)sh->vocab, k, plan.splits, plan.chunk, conf, idx, partial);
}

// The plan's split records go to `ws` (at least traj_confidence_topk_workspace_size() bytes);
// without one the rows run unsplit.
template <typename T, int K>
traj_status launch_topk_k(const void* logits, const traj_logits_shape* sh, int k, float* conf, int32_t* idx,
                          void* ws, size_t ws_bytes, hipStream_t st) {
    TopkPlan plan = plan_conf_topk(sh->rows, sh->vocab, VecOf<T>::n);
    const size_t need = (size_t)sh->rows * plan.splits * kTopkRecord * sizeof(float);
    if (plan.splits > 1 && (ws == nullptr || ws_bytes < need || !aligned16(ws))) {
        plan.splits = 1;
        plan.chunk = (int)sh->vocab;
    }
    if (sh->rows == 0) return TRAJ_OK;
    float* partial = plan.splits > 1 ? static_cast<float*>(ws) : nullptr;
    const T* lg = static_cast<const T*>(logits);
    if (plan.threads == 64) {
        launch_conf_kernel<T, K, 64, 2, 3>(lg, sh, k, plan, conf, idx, partial, st);
    } else if (plan.threads == 256) {
        launch_conf_kernel<T, K, 256, 2, 2>(lg, sh, k, plan, conf, idx, partial, st);
    } else if (plan.unroll == 4) {
        launch_conf_kernel<T, K, 512, 4, 2>(lg, sh, k, plan, conf, idx, partial, st);
    } else {
        launch_conf_kernel<T, K, 512, 2, 2>(lg, sh, k, plan, conf, idx, partial, st);
    }
    if (plan.splits > 1) {
        hipLaunchKernelGGL((conf_topk_merge_kernel<K>), dim3((unsigned)sh->rows), dim3(64), 0, st, partial,
                           (int)sh->rows, plan.splits, k, conf, idx);
    }
    return launched();
}

template <typename T>
traj_status launch_topk(const void* logits, const traj_logits_shape* sh, int k, float* conf, int32_t* idx,
                        void* ws, size_t ws_bytes, hipStream_t st) {
    switch (k) {
        case 1: return launch_topk_k<T, 1>(logits, sh, k, conf, idx, ws, ws_bytes, st);
        case 2: return launch_topk_k<T, 2>(logits, sh, k, conf, idx, ws, ws_bytes, st);
        case 3:
        case 4: return launch_topk_k<T, 4>(logits, sh, k, conf, idx, ws, ws_bytes, st);
        default: return launch_topk_k<T, 8>(logits, sh, k, conf, idx, ws, ws_bytes, st);
    }
}

// ------------------------------------------------------------------ verification layer
// Tilings of the projection GEMM with the figures its plan is made from, measured on an MI355X:
// the microseconds one 64-wide k step takes with a workgroup on every CU, the rate in TB/s at which the
// weights stream when they bound the call, the microseconds to fill and drain the stage ring, and those that
// a further round of workgroups takes beside its steps (its own fill and stores, measured with K = 64 .. 512;
// the step times, from kGemmLongSteps steps a round, hold them: without them 145 x 72 x 16832 ran on four
// rounds of 64 x 64 tiles, 13.0 us against 6.7).  Large tiles do more arithmetic per step and byte, small ones
// fill the chip where M x N is small.
// The figures are those with which the plan comes nearest to the fastest tiling and split of 326 products of 1
// .. 1024 rows (weights from HBM, every split; among them the projections and heads of 8B-class layers) and 180
// products of 3 .. 32768 rows: 0.8% and 1.1% above it on the geometric mean, at worst 12% and 18%.  With earlier
// figures, from one and two rounds of long K, few rows split too little: 128 x 12288 x 4096 34.0 us, 31.3 now.
struct GemmTiling {
    int bm, bn, threads;
    float step_us, stream, fill_us, round_us;
    void (*kernel[2][4])(GemmParams);  // [at most two row tiles][GemmEpilogue]
};
// At most two row tiles share a W tile, at about the same time: the 64-row tilings then load W
// non-temporally (gate / up of 64 / 96 / 128 rows 47.6 / 52.3 / 55.8 -> 46.5 / 51.0 / 54.7 us, down 33.7 / 36.5 /
// 35.4 -> 32.9 / 36.2 / 35.0).  Where more share it the hint costs the others' reads (256 x 128 tiles with it
// / without: 6100 x 2960 x 6760 308 / 250 us, 9904 x 728 x 6672 175 / 146).
#define TRAJ_RING_KERNELS(BM, BN, WM, WN, S, KC, NT)                                                                \
    {gemm_ring_kernel<BM, BN, WM, WN, S, KC, NT, kEpiStore>, gemm_ring_kernel<BM, BN, WM, WN, S, KC, NT, kEpiAccumulate>, \
     gemm_ring_kernel<BM, BN, WM, WN, S, KC, NT, kEpiPartial>, gemm_ring_kernel<BM, BN, WM, WN, S, KC, NT, kEpiSwiglu>}
#define TRAJ_RING_TILING(BM, BN, WM, WN, S, KC, STEP, STREAM, FILL, ROUND)                                          \
    {BM, BN, WM * WN * 64, STEP, STREAM, FILL, ROUND,                                                               \
     {TRAJ_RING_KERNELS(BM, BN, WM, WN, S, KC, false), TRAJ_RING_KERNELS(BM, BN, WM, WN, S, KC, (BM == 64 && BN > 64))}}
const GemmTiling kGemmTilings[] = {
    TRAJ_RING_TILING(64, 64, 2, 2, 9, 4, 0.34f, 4.1f, 3.5f, 2.3f),
    TRAJ_RING_TILING(64, 128, 2, 2, 3, 2, 0.54f, 6.2f, 3.5f, 1.7f),
    TRAJ_RING_TILING(64, 256, 1, 4, 4, 1, 0.97f, 6.6f, 4.0f, 4.3f),
    TRAJ_RING_TILING(128, 128, 2, 2, 4, 1, 0.57f, 5.8f, 4.0f, 3.3f),
    TRAJ_RING_TILING(256, 96, 4, 1, 3, 1, 0.755f, 5.4f, 4.0f, 4.4f),
    TRAJ_RING_TILING(256, 128, 4, 2, 3, 1, 0.93f, 5.0f, 4.0f, 5.0f),
    TRAJ_RING_TILING(128, 192, 2, 2, 4, 1, 0.855f, 5.4f, 4.0f, 4.6f),
    TRAJ_RING_TILING(192, 128, 2, 2, 4, 1, 0.71f, 4.9f, 4.5f, 4.7f),
    TRAJ_RING_TILING(128, 256, 2, 4, 3, 1, 0.92f, 6.6f, 5.0f, 5.0f),
    TRAJ_RING_TILING(192, 192, 2, 2, 3, 1, 0.95f, 5.2f, 4.5f, 6.3f),
    {kG2BM, kG2BN, kG2Threads, 1.40f, 5.5f, 3.5f, 8.7f,
     {{gemm_tile256_kernel<kEpiStore>, gemm_tile256_kernel<kEpiAccumulate>, nullptr, gemm_tile256_kernel<kEpiSwiglu>},
      {gemm_tile256_kernel<kEpiStore>, gemm_tile256_kernel<kEpiAccumulate>, nullptr, gemm_tile256_kernel<kEpiSwiglu>}}},
};
#undef TRAJ_RING_KERNELS
#undef TRAJ_RING_TILING

constexpr int kGemmCus = 256;           // workgroups the chip runs at a time
constexpr double kGemmLongSteps = 64.0;
constexpr int64_t kGemmMinSplitK = 512;
// SwiGLU goes into the GEMM's own epilogue from this many rows on: there the projection is bound
// by the matrix cores and the gate / up values' round trip through memory costs as much as it
// saves (768 rows: 147 us against 134 + 11) or more (32768 rows).  With fewer rows the weights'
// streaming bounds it and the two half-width column segments per row cost more than the separate
// launch (224 rows: 67 against 57 + 5 us; 64 rows: 48 against 42 + 5).
constexpr int64_t kSwigluFuseMinRows = 512;

struct GemmPlan {
    const GemmTiling* tiling;
    int64_t tiles_m, tiles_n;
    int splits, k_split;
};

// The tiling and K split (into at most max_splits ranges) with the least estimated time: rounds of
// workgroups over the CUs times their steps, but at least the weights' streaming time, and for a split the
// second launch and its partial products' traffic (written and read).  A split's reduction applies SwiGLU at no
// cost; without one it is a launch of its own below kSwigluFuseMinRows.
GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, bool swiglu, int64_t max_splits) {
    GemmPlan best{};
    double best_us = 0.0;
    const int64_t steps = (K + kGemmBK - 1) / kGemmBK;
    for (const GemmTiling& g : kGemmTilings) {
        const int64_t tm = (M + g.bm - 1) / g.bm, tn = (N + g.bn - 1) / g.bn;
        const double stream_us = (double)K * (double)N * 2e-6 / g.stream;
        for (int s = 1; s <= kGemmMaxSplits; ++s) {
            if (s > 1 && (s > max_splits || g.kernel[0][kEpiPartial] == nullptr || K / s < kGemmMinSplitK || tm * tn * s > kGemmCus)) break;
            const int64_t split_steps = (steps + s - 1) / s;
            if ((steps + split_steps - 1) / split_steps != s) continue;  // the same as a smaller s
            const double rounds = (double)((tm * tn * s + kGemmCus - 1) / kGemmCus);
            const double fills = (rounds - 1.0) * std::max(0.0, 1.0 - (double)split_steps / kGemmLongSteps) * g.round_us;
            double us = std::max(rounds * (double)split_steps * g.step_us + fills, stream_us) + g.fill_us;
            if (s > 1) us += 3.2 + 0.27 * s + (double)s * (double)M * (double)N * 8.0 / 7.1e6;
            if (s == 1 && swiglu && M < kSwigluFuseMinRows) us += 6.0;
            if (best.tiling == nullptr || us < best_us) {
                best = GemmPlan{&g, tm, tn, s, s > 1 ? (int)(split_steps * kGemmBK) : 0};
                best_us = us;
            }
        }
    }
    return best;
}

bool gemm_sizes_ok(int64_t M, int64_t N, int64_t K) { return M >= 1 && N >= 8 && K >= 8 && K <= kGemmMaxK && N <= kGemmMaxN; }

size_t partial_bytes(int64_t M, int64_t N) { return (size_t)M * (size_t)N * sizeof(float); }  // of one k range

// fp32 partial products of a split GEMM (0 when the shape is not split)
size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (!gemm_sizes_ok(M, N, K)) return 0;
    const int splits = plan_gemm(M, N, K, false, kGemmMaxSplits).splits;
    return splits > 1 ? splits * partial_bytes(M, N) : 0;
}

// Partial products of as many k ranges as 128 x 128 tiles leave CUs for (0: none).  Fixed by the sizes: what
// traj_linear reports is never below it and what it accepts never above, so that a workspace which served a
// set of shapes goes on to serve them when the plan's figures change.
size_t gemm_fixed_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (!gemm_sizes_ok(M, N, K)) return 0;
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    int64_t splits = std::min<int64_t>(kGemmCus / tiles, std::min<int64_t>(K / kGemmMinSplitK, kGemmMaxSplits));
    if (splits <= 1) return 0;
    const int64_t steps = (K + kGemmBK - 1) / kGemmBK, split_steps = (steps + splits - 1) / splits;
    splits = (steps + split_steps - 1) / split_steps;
    return splits * partial_bytes(M, N);
}

// Scratch of the gate / up projection with SwiGLU: the partial products, or the [M, N] gate / up
// values where SwiGLU is a launch of its own.
size_t gemm_swiglu_workspace_bytes(int64_t M, int64_t N, int64_t K) {
    if (!gemm_sizes_ok(M, N, K)) return 0;
    const int splits = plan_gemm(M, N, K, true, kGemmMaxSplits).splits;
    if (splits > 1) return splits * partial_bytes(M, N);
    return M < kSwigluFuseMinRows ? (size_t)M * (size_t)N * sizeof(uint16_t) : 0;
}

// D[M,N] = A[M,K] W[K,N] (+ D with kEpiAccumulate), or with kEpiSwiglu D[M,N/2] = silu(gate) * up
// of the product's [gate | up] columns; bf16 row-major, fp32 accumulation.  `ws` holds the split-K
// partials: the plan splits into as many ranges as fit it (null: none), and SwiGLU stays in the epilogue
// where the gate / up values don't fit.
// With `pending` a split leaves its sum to the caller: *pending is the number of partial products in
// ws (1: D holds the result).
traj_status gemm(const uint16_t* A, const uint16_t* W, uint16_t* D, int64_t M, int64_t N, int64_t K, GemmEpilogue epi,
                 void* ws, size_t ws_bytes, hipStream_t st, int* pending = nullptr) {
    if (M < 1 || N < 8 || K < 8 || N % 8 != 0 || K % 8 != 0) return TRAJ_E_SHAPE;
    if (M > INT_MAX - kG2BM) return TRAJ_E_SHAPE;
    if (K > kGemmMaxK || N > kGemmMaxN) return TRAJ_E_UNSUPPORTED;  // 32-bit buffer offsets
    if (!aligned16(A) || !aligned16(W) || !aligned16(D)) return TRAJ_E_SHAPE;
    if (ws == nullptr || !aligned16(ws)) ws_bytes = 0;
    const bool swiglu = epi == kEpiSwiglu;
    const GemmPlan g = plan_gemm(M, N, K, swiglu, (int64_t)(ws_bytes / partial_bytes(M, N)));
    // SwiGLU as its own launch
    const bool apart = swiglu && g.splits == 1 && M < kSwigluFuseMinRows && ws_bytes >= (size_t)M * (size_t)N * sizeof(uint16_t);
    const dim3 grid((unsigned)(g.tiles_m * g.tiles_n), (unsigned)g.splits);
    const GemmParams p{A, W, apart ? static_cast<uint16_t*>(ws) : D, (int)M, (int)N, (int)K, (int)g.tiles_m, (int)g.tiles_n,
                       g.splits > 1 ? static_cast<float*>(ws) : nullptr, g.k_split};
    hipLaunchKernelGGL(g.tiling->kernel[g.tiles_m <= 2][g.splits > 1 ? kEpiPartial : apart ? kEpiStore : epi], grid, dim3(g.tiling->threads), 0,
                       st, p);
    const traj_status rs = launched();
    if (pending != nullptr) *pending = g.splits;
    if (rs != TRAJ_OK || (g.splits == 1 && !apart) || (g.splits > 1 && pending != nullptr)) return rs;
    const int64_t chunks = M * (swiglu ? N / 2 : N) / 8;
    const dim3 rgrid((unsigned)std::min<int64_t>((chunks + 255) / 256, 4096));
    if (apart) {
        hipLaunchKernelGGL(swiglu_kernel, rgrid, dim3(256), 0, st, static_cast<const uint16_t*>(ws), D, (int)M, (int)N);
    } else {
        auto reduce = swiglu                  ? gemm_split_reduce_kernel<kEpiSwiglu>
                      : epi == kEpiAccumulate ? gemm_split_reduce_kernel<kEpiAccumulate>
                                              : gemm_split_reduce_kernel<kEpiStore>;
        hipLaunchKernelGGL(reduce, rgrid, dim3(256), 0, st, static_cast<const float*>(ws), g.splits, D, (int)M, (int)N);
    }
    return launched();
}

size_t align256(size_t n) { return (n + 255) / 256 * 256; }

// The intermediates' places in a layer's workspace.  What follows them is the projections' scratch: the
// layer runs with any size of it (none: nothing is split), `total` holds what its plans would use.
struct LayerPlan {
    size_t xn, qkv, q, kd, vd, a, act, split, total;
};

LayerPlan plan_layer(const traj_attn_shape* sh, const traj_layer_dims* dm) {
    const size_t T = (size_t)sh->B * sh->N * sh->L;
    LayerPlan p{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align256(bytes);
        return at;
    };
    p.xn = take(T * dm->hidden * 2);
    p.qkv = take(T * (size_t)(sh->Hq + 2 * sh->Hkv) * sh->D * 2);
    p.q = take(T * (size_t)sh->Hq * sh->D * 2);
    p.kd = take(T * (size_t)sh->Hkv * sh->D * 2);
    p.vd = take(T * (size_t)sh->Hkv * sh->D * 2);
    p.a = take(T * (size_t)sh->Hq * sh->D * 2);
    p.act = take(T * (size_t)dm->inter * 2);
    const int64_t hid = dm->hidden, qkv_w = (int64_t)(sh->Hq + 2 * sh->Hkv) * sh->D;
    const size_t scratch = std::max(std::max(gemm_workspace_bytes(T, qkv_w, hid), gemm_workspace_bytes(T, hid, (int64_t)sh->Hq * sh->D)),
                                    std::max(gemm_swiglu_workspace_bytes(T, 2 * (int64_t)dm->inter, hid),
                                             gemm_workspace_bytes(T, hid, dm->inter)));
    p.split = take(scratch);
    p.total = off;
    return p;
}

traj_status check_layer(const traj_attn_shape* sh, const traj_layer_dims* dm) {
    if (sh == nullptr || dm == nullptr) return TRAJ_E_NULL;
    const traj_status st = check_attn(sh);
    if (st != TRAJ_OK) return st;
    if (dm->hidden != sh->Hq * sh->D || dm->hidden % 8 != 0 || dm->inter < 8 || dm->inter % 8 != 0) return TRAJ_E_SHAPE;
    if (!(dm->rms_eps >= 0.f) || !(dm->rope_theta > 0.f)) return TRAJ_E_ARG;
    return TRAJ_OK;
}

traj_status check_weights(const void* x, const traj_layer_weights* w) {
    if (w == nullptr || w->attn_norm == nullptr || w->w_qkv == nullptr || w->w_o == nullptr ||
        w->mlp_norm == nullptr || w->w_gate_up == nullptr || w->w_down == nullptr)
        return TRAJ_E_NULL;
    if (!aligned16(x) || !aligned16(w->attn_norm) || !aligned16(w->mlp_norm) || !aligned16(w->w_qkv) ||
        !aligned16(w->w_o) || !aligned16(w->w_gate_up) || !aligned16(w->w_down))
        return TRAJ_E_SHAPE;
    return TRAJ_OK;
}

// The refresh's layer runs over B whole sequences of T = S + L tokens; `as` receives the
// equivalent attention shape (one "draft" of T tokens, the sequence's own K / V as its cache).
traj_status check_refresh(const traj_refresh_shape* sh, const traj_layer_dims* dm, traj_attn_shape* as) {
    if (sh == nullptr || dm == nullptr) return TRAJ_E_NULL;
    if (sh->B < 1 || sh->S < 0 || sh->L < 1 || (int64_t)sh->S + sh->L > 0x7fffffff / 2) return TRAJ_E_SHAPE;
    *as = traj_attn_shape{sh->B, 1, sh->S + sh->L, sh->Hq, sh->Hkv, sh->D, sh->S + sh->L, sh->scale};
    return check_layer(as, dm);
}

// Cache-only attention: every query row of q [B, T, Hq, D] attends to the S keys of k / v
// [B, S, Hkv, D] (the attention kernel with empty draft visible sets, N = 1, L = T).
traj_status attn_cache_only(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* out, int B, int T,
                            int S, int Hq, int Hkv, int D, float scale_in, hipStream_t s) {
    const traj_attn_shape sh{B, 1, T, Hq, Hkv, D, S, scale_in};
    const traj_status st = check_attn(&sh);
    if (st != TRAJ_OK) return st;
    AttnParams p{};
    p.q = q;
    p.kc = k;
    p.vc = v;
    p.kd = k;  // never read: no draft is visible
    p.vd = v;
    p.parent = nullptr;
    p.peers = nullptr;
    p.out = out;
    p.B = B;
    p.N = 1;
    p.L = T;
    p.Hq = Hq;
    p.Hkv = Hkv;
    p.S = S;
    p.group = Hq / Hkv;
    p.rows_per_group = p.group * T;
    const int rb = (p.rows_per_group + 31) / 32;
    p.wg_per_group = (rb + kAttnWaves - 1) / kAttnWaves;
    const int64_t nwg = (int64_t)B * Hkv * p.wg_per_group;
    if (nwg > 0x7fffffff) return TRAJ_E_SHAPE;
    p.num_wg = (int)nwg;
    const float scale = scale_in > 0.f ? scale_in : 1.0f / std::sqrt((float)D);
    p.scale_log2 = scale * 1.4426950408889634f;
    p.drafts_visible = 0;
    return D == 128 ? launch_attn<128>(p, s) : launch_attn<64>(p, s);
}

// out = norm(x) * w over T rows; with splits > 1 x first gains the sum of the partial products.  A launch
// holds fewer than 2^32 threads, so more rows than kNormMaxRows take several (a split has far fewer).
constexpr int64_t kNormMaxRows = (1ll << 32) / 512 - 1;
template <bool SPLIT>
traj_status launch_rmsnorm(uint16_t* x, const void* w, uint16_t* out, int64_t T, int hidden, float eps, const float* partial,
                           int splits, hipStream_t s) {
    const int nv = hidden / 8;
    auto kernel = nv <= 256    ? rmsnorm_kernel<256, 1, SPLIT>
                  : nv <= 512  ? rmsnorm_kernel<512, 1, SPLIT>
                  : nv <= 1024 ? rmsnorm_kernel<512, 2, SPLIT>
                               : rmsnorm_kernel<512, 0, SPLIT>;
    for (int64_t t = 0; t < T; t += kNormMaxRows) {
        const dim3 grid((unsigned)std::min<int64_t>(T - t, kNormMaxRows));
        hipLaunchKernelGGL(kernel, grid, dim3(nv <= 256 ? 256 : 512), 0, s, x + t * hidden, static_cast<const uint16_t*>(w),
                           out + t * hidden, hidden, eps, partial, splits);
        const traj_status st = launched();
        if (st != TRAJ_OK) return st;
    }
    return TRAJ_OK;
}

traj_status rmsnorm(uint16_t* x, const void* w, uint16_t* out, int64_t T, int hidden, float eps, const float* partial, int splits,
                    hipStream_t s) {
    return splits > 1 ? launch_rmsnorm<true>(x, w, out, T, hidden, eps, partial, splits, s)
                      : launch_rmsnorm<false>(x, w, out, T, hidden, eps, nullptr, 1, s);
}

// One pre-norm decoder layer over T packed tokens (x [T, hidden], updated in place).  The rotary
// position of token t is pos0[t / rope_nl] + t % rope_l (pos0 may be null = 0); `attend` runs
// between the rotary split and the O projection: it reads the q / k / v rows and writes the
// attention output a [T, Hq D].
template <typename Attend>
traj_status run_layer(uint16_t* xs, const traj_layer_weights* w, const traj_layer_dims* dims, int64_t T, int Hq,
                      int Hkv, int D, const int32_t* pos0, int rope_nl, int rope_l, const CacheRows& cache,
                      const LayerPlan& plan, char* ws, size_t ws_bytes, hipStream_t s, Attend attend) {
    auto buf = [&](size_t off) { return reinterpret_cast<uint16_t*>(ws + off); };
    const int hidden = dims->hidden, inter = dims->inter;
    const int qkv_w = (Hq + 2 * Hkv) * D;
    void* split = ws + plan.split;
    const size_t split_bytes = ws_bytes - plan.split;
    traj_status st;
    const float* partial = static_cast<const float*>(split);
    // attention block
    if ((st = rmsnorm(xs, w->attn_norm, buf(plan.xn), T, hidden, dims->rms_eps, nullptr, 1, s)) != TRAJ_OK) return st;
    int pending = 1;  // partial products the next kernel sums
    if ((st = gemm(buf(plan.xn), static_cast<const uint16_t*>(w->w_qkv), buf(plan.qkv), T, qkv_w, hidden, kEpiStore, split,
                   split_bytes, s, &pending)) != TRAJ_OK)
        return st;
    // few tokens: a chunk pair per thread, so that no thread waits on memory twice
    const unsigned rope_y = T < 1024 ? (unsigned)((qkv_w / 16 + kLayerThreads - 1) / kLayerThreads) : 1u;
    hipLaunchKernelGGL(pending > 1 ? rope_split_kernel<true> : rope_split_kernel<false>, dim3((unsigned)T, rope_y),
                       dim3(kLayerThreads), 0, s, buf(plan.qkv), partial, pending, pos0, buf(plan.q), buf(plan.kd),
                       buf(plan.vd), rope_nl, rope_l, Hq, Hkv, D, std::log2(dims->rope_theta), cache);
    if ((st = launched()) != TRAJ_OK) return st;
    if ((st = attend(buf(plan.q), buf(plan.kd), buf(plan.vd), buf(plan.a))) != TRAJ_OK) return st;
    if ((st = gemm(buf(plan.a), static_cast<const uint16_t*>(w->w_o), xs, T, hidden, (int64_t)Hq * D, kEpiAccumulate, split,
                   split_bytes, s, &pending)) != TRAJ_OK)
        return st;
    // MLP block
    if ((st = rmsnorm(xs, w->mlp_norm, buf(plan.xn), T, hidden, dims->rms_eps, partial, pending, s)) != TRAJ_OK) return st;
    if ((st = gemm(buf(plan.xn), static_cast<const uint16_t*>(w->w_gate_up), buf(plan.act), T, 2 * (int64_t)inter, hidden,
                   kEpiSwiglu, split, split_bytes, s)) != TRAJ_OK)
        return st;
    return gemm(buf(plan.act), static_cast<const uint16_t*>(w->w_down), xs, T, hidden, inter, kEpiAccumulate, split, split_bytes, s);
}

}  // namespace

extern "C" {

size_t traj_verify_attn_workspace_size(const traj_attn_shape* shape) {
    (void)shape;
    return 0;  // the attention kernels use no scratch memory; the workspace argument is reserved
}

traj_status traj_verify_attn(const void* q, const void* k_cache, const void* v_cache, const void* k_draft,
                             const void* v_draft, const int32_t* draft_parent, void* out,
                             const traj_attn_shape* shape, void* workspace, size_t workspace_bytes, void* stream) {
    return traj_verify_attn_peers(q, k_cache, v_cache, k_draft, v_draft, draft_parent, nullptr, out, shape,
                                  workspace, workspace_bytes, stream);
}

traj_status traj_verify_attn_peers(const void* q, const void* k_cache, const void* v_cache, const void* k_draft,
                                   const void* v_draft, const int32_t* draft_parent, const uint64_t* draft_peers,
                                   void* out, const traj_attn_shape* shape, void* workspace, size_t workspace_bytes,
                                   void* stream) {
    (void)workspace;
    (void)workspace_bytes;
    return verify_attn(q, k_cache, v_cache, k_draft, v_draft, draft_parent, draft_peers, out, shape, false, as_stream(stream));
}

size_t traj_confidence_topk_workspace_size(const traj_logits_shape* shape, int32_t k) {
    if (shape == nullptr || check_logits(shape, k) != TRAJ_OK) return 0;
    const TopkPlan plan = plan_conf_topk(shape->rows, shape->vocab, vec_of(shape->dtype));
    if (plan.splits <= 1) return 0;
    return (size_t)shape->rows * plan.splits * kTopkRecord * sizeof(float);
}

traj_status traj_confidence_topk(const void* logits, int32_t k, float* conf, int32_t* idx,
                                 const traj_logits_shape* shape, void* workspace, size_t workspace_bytes,
                                 void* stream) {
    if (shape == nullptr) return TRAJ_E_NULL;
    traj_status st = check_logits(shape, k);
    if (st != TRAJ_OK) return st;
    if (shape->rows == 0) return TRAJ_OK;  // nothing to do; pointers may be NULL
    if (logits == nullptr || conf == nullptr || idx == nullptr) return TRAJ_E_NULL;
    if (workspace != nullptr && !aligned16(workspace)) return TRAJ_E_WORKSPACE;
    const size_t need = traj_confidence_topk_workspace_size(shape, k);
    if (workspace != nullptr && workspace_bytes > 0 && workspace_bytes < need) return TRAJ_E_WORKSPACE;
    hipStream_t s = as_stream(stream);
    if (shape->dtype == TRAJ_BF16) return launch_topk<uint16_t>(logits, shape, k, conf, idx, workspace, workspace_bytes, s);
    return launch_topk<float>(logits, shape, k, conf, idx, workspace, workspace_bytes, s);
}

traj_status traj_confidence_topk_noalloc(const void* logits, int32_t k, float* conf, int32_t* idx,
                                         const traj_logits_shape* shape, void* stream) {
    if (shape == nullptr) return TRAJ_E_NULL;
    traj_status st = check_logits(shape, k);
    if (st != TRAJ_OK) return st;
    if (shape->rows == 0) return TRAJ_OK;
    if (logits == nullptr || conf == nullptr || idx == nullptr) return TRAJ_E_NULL;
    const size_t need = traj_confidence_topk_workspace_size(shape, k);
    if (need > (size_t)TRAJ_TOPK_SCRATCH_BYTES) return TRAJ_E_WORKSPACE;  // split records beyond the fixed scratch
    void* ws = nullptr;
    if (need > 0 && (st = device_scratch(&ws)) != TRAJ_OK) return st;
    hipStream_t s = as_stream(stream);
    if (shape->dtype == TRAJ_BF16) return launch_topk<uint16_t>(logits, shape, k, conf, idx, ws, need, s);
    return launch_topk<float>(logits, shape, k, conf, idx, ws, need, s);
}

traj_status traj_accept(const float* conf, const int32_t* idx, const traj_drafts* drafts, float threshold,
                        const traj_accepted* accepted, void* stream) {
    if (drafts == nullptr || accepted == nullptr || conf == nullptr || idx == nullptr) return TRAJ_E_NULL;
    if (drafts->tokens == nullptr || drafts->parent == nullptr || drafts->committed == nullptr ||
        drafts->conf0 == nullptr || drafts->idx0 == nullptr)
        return TRAJ_E_NULL;
    if (accepted->leaf == nullptr || accepted->on_path == nullptr || accepted->n_accepted == nullptr ||
        accepted->out_tokens == nullptr || accepted->hi == nullptr)
        return TRAJ_E_NULL;
    if (drafts->B < 1 || drafts->N < 1 || drafts->N > kMaxDrafts || drafts->L < 1 || drafts->L > kMaxBlock)
        return TRAJ_E_SHAPE;
    if (drafts->k < 1 || drafts->k > 8) return TRAJ_E_ARG;
    if (drafts->mode < TRAJ_MODE_EXACT || drafts->mode > TRAJ_MODE_TOPK) return TRAJ_E_ARG;
    if (drafts->traversal != TRAJ_GREEDY && drafts->traversal != TRAJ_LONGEST) return TRAJ_E_ARG;
    if (!(threshold == threshold)) return TRAJ_E_ARG;
    AcceptParams p{};
    p.conf = conf;
    p.idx = idx;
    p.tokens = drafts->tokens;
    p.parent = drafts->parent;
    p.committed = drafts->committed;
    p.conf0 = drafts->conf0;
    p.idx0 = drafts->idx0;
    p.leaf = accepted->leaf;
    p.on_path = accepted->on_path;
    p.n_accepted = accepted->n_accepted;
    p.out_tokens = accepted->out_tokens;
    p.hi = accepted->hi;
    p.B = drafts->B;
    p.N = drafts->N;
    p.L = drafts->L;
    p.k = drafts->k;
    p.mode = drafts->mode;
    p.traversal = drafts->traversal;
    p.tau = threshold;
    hipLaunchKernelGGL(accept_kernel, dim3(p.B), dim3(kAcceptThreads), 0, as_stream(stream), p);
    return launched();
}

traj_status traj_interblock_trigger(const int32_t* state, const float* conf, int32_t B, int32_t L, int32_t k,
                                    float threshold, uint8_t* trigger, float* c_cur, float* c_next, void* stream) {
    if (state == nullptr || conf == nullptr || trigger == nullptr) return TRAJ_E_NULL;
    if (B < 1 || L < 1 || L > kTriggerMaxBlock) return TRAJ_E_SHAPE;
    if (k < 1 || k > 8 || !(threshold == threshold)) return TRAJ_E_ARG;
    TriggerParams p{state, conf, trigger, c_cur, c_next, B, L, k, threshold};
    hipLaunchKernelGGL(interblock_trigger_kernel, dim3(B), dim3(64), 0, as_stream(stream), p);
    return launched();
}

traj_status traj_joint_peers(int32_t B, int32_t n_cur, int32_t n_next, const int32_t* root_cur,
                             const int32_t* root_next, uint64_t* peers, void* stream) {
    if (peers == nullptr) return TRAJ_E_NULL;
    if (B < 1 || n_cur < 1 || n_next < 1 || n_cur + n_next > 64) return TRAJ_E_SHAPE;
    const int64_t total = (int64_t)B * (n_cur + n_next);
    if (total > ((int64_t)1 << 31) - 256) return TRAJ_E_SHAPE;
    static_assert(kDevBadRoot == TRAJ_DEV_BAD_ROOT, "device status bit");
    const JointPeersParams p{root_cur, root_next, peers, B, n_cur, n_next};
    hipLaunchKernelGGL(joint_peers_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, as_stream(stream), p);
    return launched();
}

int32_t traj_tree_max_nodes(const traj_tree_shape* sh) {
    if (sh == nullptr || sh->B < 1 || sh->L < 1 || sh->L > kTreeMaxBlock || sh->k < 1 || sh->k > kTreeMaxK ||
        sh->branch < 1 || sh->branch > sh->k || sh->branch_deep < 1 || sh->branch_deep > sh->k || sh->width < 1 ||
        sh->depth < 0 || sh->n_prev < 0 || (sh->full != 0 && sh->full != 1))
        return -1;
    int64_t total = 1, cnt = 0;
    const int levels = sh->depth < sh->L ? sh->depth : sh->L;
    for (int l = 1; l <= levels; ++l) {
        const int64_t w = sh->full ? sh->width : (sh->width - l + 1 > 1 ? sh->width - l + 1 : 1);
        const int64_t gen = l == 1 ? sh->branch : cnt * sh->branch_deep;
        cnt = gen < w ? gen : w;
        total += cnt;
        if (total > 0x7fffffff) return -1;
    }
    return (int32_t)total;
}

traj_status traj_build_tree(const int32_t* state, const int32_t* leaf, const float* conf, const int32_t* idx,
                            const float* conf0, const int32_t* idx0, const traj_tree_shape* shape, float threshold,
                            int32_t* tokens, int32_t* parent, int32_t* n_nodes, float* score, float* conf_next,
                            int32_t* idx_next, void* stream) {
    if (shape == nullptr || state == nullptr || conf0 == nullptr || idx0 == nullptr || tokens == nullptr ||
        parent == nullptr || n_nodes == nullptr)
        return TRAJ_E_NULL;
    if (leaf != nullptr && shape->n_prev > 0 && (conf == nullptr || idx == nullptr)) return TRAJ_E_NULL;
    if ((conf_next == nullptr) != (idx_next == nullptr)) return TRAJ_E_NULL;
    if (shape->k < 1 || shape->k > kTreeMaxK || shape->branch < 1 || shape->branch > shape->k ||
        shape->branch_deep < 1 || shape->branch_deep > shape->k || (shape->full != 0 && shape->full != 1))
        return TRAJ_E_ARG;
    if (!(threshold == threshold)) return TRAJ_E_ARG;
    const int32_t need = traj_tree_max_nodes(shape);
    if (need < 0 || shape->n_max < need || shape->n_max > kTreeMaxNodes) return TRAJ_E_SHAPE;
    TreeParams p{};
    p.state = state;
    p.leaf = leaf;
    p.conf = conf;
    p.idx = idx;
    p.conf0 = conf0;
    p.idx0 = idx0;
    p.tokens = tokens;
    p.parent = parent;
    p.n_nodes = n_nodes;
    p.score = score;
    p.conf_next = conf_next;
    p.idx_next = idx_next;
    p.B = shape->B;
    p.L = shape->L;
    p.k = shape->k;
    p.n_prev = leaf != nullptr ? shape->n_prev : 0;
    p.width = shape->width;
    p.depth = shape->depth;
    p.branch = shape->branch;
    p.branch_deep = shape->branch_deep;
    p.full = shape->full;
    p.n_max = shape->n_max;
    p.tau = threshold;
    hipLaunchKernelGGL(build_tree_kernel, dim3(p.B), dim3(kTreeThreads), 0, as_stream(stream), p);
    return launched();
}

size_t traj_verify_layer_workspace_size(const traj_attn_shape* shape, const traj_layer_dims* dims) {
    if (check_layer(shape, dims) != TRAJ_OK) return 0;
    return plan_layer(shape, dims).total;
}

traj_status traj_verify_layer(void* x, const traj_layer_weights* w, const traj_layer_dims* dims, const void* k_cache,
                              const void* v_cache, const int32_t* draft_parent, const int32_t* pos0,
                              const traj_attn_shape* shape, void* workspace, size_t workspace_bytes, void* stream) {
    traj_status st = check_layer(shape, dims);
    if (st != TRAJ_OK) return st;
    if (x == nullptr || draft_parent == nullptr || workspace == nullptr) return TRAJ_E_NULL;
    if ((st = check_weights(x, w)) != TRAJ_OK) return st;
    if (shape->S > 0 && (k_cache == nullptr || v_cache == nullptr)) return TRAJ_E_NULL;
    const LayerPlan plan = plan_layer(shape, dims);
    if (workspace_bytes < plan.split || reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return TRAJ_E_WORKSPACE;
    const int64_t T = (int64_t)shape->B * shape->N * shape->L;
    // The cache was last read a forward pass ago: where the layers' weights since then have displaced it
    // from the last-level cache it streams from HBM, and the attention's chain of steps waits for each
    // stage unless the cache is read ahead (a cache that is still near costs the call 1 us more).
    const bool warm = ((int64_t)dims->hidden * (shape->Hq + 2 * shape->Hkv + shape->Hq) * shape->D +
                       3 * (int64_t)dims->hidden * dims->inter) * 2 >= kAttnWarmLayerBytes;
    // every draft's token p sits at position pos0[b] + p
    return run_layer(static_cast<uint16_t*>(x), w, dims, T, shape->Hq, shape->Hkv, shape->D, pos0,
                     shape->N * shape->L, shape->L, CacheRows{}, plan, static_cast<char*>(workspace), workspace_bytes,
                     as_stream(stream),
                     [&](const uint16_t* q, const uint16_t* kd, const uint16_t* vd, uint16_t* a) {
                         return verify_attn(q, k_cache, v_cache, kd, vd, draft_parent, nullptr, a, shape, warm, as_stream(stream));
                     });
}

size_t traj_refresh_layer_workspace_size(const traj_refresh_shape* shape, const traj_layer_dims* dims) {
    traj_attn_shape as{};
    if (check_refresh(shape, dims, &as) != TRAJ_OK) return 0;
    return plan_layer(&as, dims).total;
}

traj_status traj_refresh_layer(void* x, const traj_layer_weights* w, const traj_layer_dims* dims,
                               const int32_t* block_start, void* k_cache, void* v_cache,
                               const traj_refresh_shape* shape, void* workspace, size_t workspace_bytes, void* stream) {
    traj_attn_shape as{};
    traj_status st = check_refresh(shape, dims, &as);
    if (st != TRAJ_OK) return st;
    if (x == nullptr || block_start == nullptr || workspace == nullptr) return TRAJ_E_NULL;
    if ((st = check_weights(x, w)) != TRAJ_OK) return st;
    if (shape->S > 0 && (k_cache == nullptr || v_cache == nullptr)) return TRAJ_E_NULL;
    if (shape->S > 0 && (!aligned16(k_cache) || !aligned16(v_cache))) return TRAJ_E_SHAPE;
    const LayerPlan plan = plan_layer(&as, dims);
    if (workspace_bytes < plan.split || reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return TRAJ_E_WORKSPACE;
    const int Tseq = shape->S + shape->L;
    const int64_t T = (int64_t)shape->B * Tseq;
    hipStream_t s = as_stream(stream);
    // positions 0 .. T - 1 of each sequence, the rows outside the block also to the cache; attention
    // over the sequence's own K / V (the kernel's cache-only mode)
    const CacheRows cache{block_start, shape->S > 0 ? static_cast<uint16_t*>(k_cache) : nullptr,
                          static_cast<uint16_t*>(v_cache), shape->S, shape->L};
    return run_layer(static_cast<uint16_t*>(x), w, dims, T, shape->Hq, shape->Hkv, shape->D, nullptr, Tseq, Tseq, cache,
                     plan, static_cast<char*>(workspace), workspace_bytes, s,
                     [&](const uint16_t* q, const uint16_t* kd, const uint16_t* vd, uint16_t* a) -> traj_status {
                         return attn_cache_only(q, kd, vd, a, shape->B, Tseq, Tseq, shape->Hq, shape->Hkv, shape->D,
                                                shape->scale, s);
                     });
}

size_t traj_linear_workspace_size(int64_t M, int64_t K, int64_t N) {
    return std::max(gemm_workspace_bytes(M, N, K), gemm_fixed_workspace_bytes(M, N, K));
}

traj_status traj_linear(const void* x, const void* w, void* y, int64_t M, int64_t K, int64_t N, int32_t accumulate,
                        void* workspace, size_t workspace_bytes, void* stream) {
    if (M < 0 || K < 8 || N < 8 || K % 8 != 0 || N % 8 != 0) return TRAJ_E_SHAPE;
    if (M == 0) return TRAJ_OK;
    if (x == nullptr || w == nullptr || y == nullptr) return TRAJ_E_NULL;
    const size_t least = std::min(gemm_workspace_bytes(M, N, K), gemm_fixed_workspace_bytes(M, N, K));
    if (workspace != nullptr && (workspace_bytes < least || !aligned16(workspace))) return TRAJ_E_WORKSPACE;
    return gemm(static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), static_cast<uint16_t*>(y), M, N, K,
                accumulate != 0 ? kEpiAccumulate : kEpiStore, workspace, workspace_bytes, as_stream(stream));
}

// For the tests: the plan of a product with all the workspace it asks for, as tile rows and columns and k
// ranges.  Not part of the interface.
void traj_test_gemm_plan(int64_t M, int64_t K, int64_t N, int32_t swiglu, int32_t plan[3]) {
    const GemmPlan g = plan_gemm(M, N, K, swiglu != 0, kGemmMaxSplits);
    plan[0] = g.tiling->bm;
    plan[1] = g.tiling->bn;
    plan[2] = g.splits;
}

const char* traj_status_string(int32_t status) {
    switch (status) {
        case TRAJ_OK: return "ok";
        case TRAJ_E_NULL: return "a required pointer is NULL";
        case TRAJ_E_SHAPE: return "a size is out of range, inconsistent or misaligned";
        case TRAJ_E_DTYPE: return "unknown element type";
        case TRAJ_E_UNSUPPORTED: return "supported by the ABI but not implemented (head_dim must be 64 or 128; one sequence's cache below 2 GiB)";
        case TRAJ_E_WORKSPACE: return "workspace too small or misaligned";
        case TRAJ_E_HIP: return "HIP runtime error";
        case TRAJ_E_ARG: return "an enumerated or scalar argument has an invalid value";
        default: return "unknown status";
    }
}

// TRAJ_SOURCE_DIGEST: sha256 of the sources and flags, stamped by the package's build script.
#ifndef TRAJ_SOURCE_DIGEST
#define TRAJ_SOURCE_DIGEST "unstamped"
#endif
const char* traj_version(void) { return "libtrajspec 0.2.0 gfx950 sources " TRAJ_SOURCE_DIGEST; }

traj_status traj_get_device_status(int32_t* host_flags, int32_t reset, void* stream) {
    if (host_flags == nullptr) return TRAJ_E_NULL;
    hipStream_t s = as_stream(stream);
    if (hipStreamSynchronize(s) != hipSuccess) return TRAJ_E_HIP;
    int32_t v = 0;
    if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_device_status), sizeof(v), 0, hipMemcpyDeviceToHost) != hipSuccess)
        return TRAJ_E_HIP;
    *host_flags = v;
    if (reset) {
        const int32_t zero = 0;
        if (hipMemcpyToSymbol(HIP_SYMBOL(g_device_status), &zero, sizeof(zero), 0, hipMemcpyHostToDevice) !=
            hipSuccess)
            return TRAJ_E_HIP;
    }
    return TRAJ_OK;
}

}  // extern "C"
