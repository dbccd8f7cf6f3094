// Trajectory-masked verification attention (Sec. 3.3) on gfx950 bf16 MFMA.
//
// Work decomposition
//   Queries of one (sequence b, K/V head g) are flattened as rows r = (hg, n, p): query head
//   g*G + hg, draft n, block position p.  A wave owns 32 consecutive rows; a workgroup of
//   4 waves owns 128 rows that all read the same K/V head, so every cache tile is staged in
//   LDS once and consumed by all four waves (cache K/V is shared by every draft).
//
// Math layout (v_mfma_f32_32x32x16_bf16, wave64)
//   Scores are computed transposed, S^T = K Q^T (32 keys x 32 queries per MFMA block): the
//   accumulator then holds one query per lane column, so the row max / row sum of the
//   online softmax is a per-lane reduction plus one exchange with lane^32 (a VALU lane
//   swap), and the output O^T = V^T P^T rescales with a per-lane scalar.  Q stays in
//   registers as the B operand.  V^T fragments come straight from a row-major V tile with
//   ds_read_b64_tr_b16.
//
// LDS layouts (contiguous rows of D elements, conflict-free for their readers)
//   K tile: the 16-byte chunk c of row r is stored at c ^ k_swz(r), so the 16 rows that
//           one fragment load reads per bank cycle hit 16 different 16-byte bank groups.
//   V tile: chunk c of row r is stored at c ^ v_rot(r) (a per-row multiple of 4), so the
//           4 rows x 64 bytes that half a wave reads with one transposing load cover all
//           64 banks once.
//   Cache tiles are filled with buffer_load_dwordx4 ... lds (16 bytes per lane straight into
//   LDS, no VGPR staging; the (b, g) slice is a buffer descriptor, the uniform row offset
//   rides in soffset and each lane keeps a 32-bit offset): each wave-wide load fills one
//   contiguous kilobyte, i.e. whole rows, and each lane fetches the global chunk that the
//   swizzle puts in its slot.  Draft tiles use global_load_lds_dwordx4 the same way.
//
// Phases per workgroup
//   0. prologue: the parent array, Q, the K rows of cache keys 0..63 and the first stage are
//      all requested before anything waits; wave 0 builds the 64-bit ancestor masks from the
//      parent array with lane shuffles.
//   1. cache, in 64-key steps: a softmax phase turns the scores of two 32-key blocks into
//      bf16 weights on the vector ALUs, then a matrix phase computes the scores of the next two
//      blocks and adds the weighted V rows of the current two (32 MFMAs back to back).  Two
//      waves of different workgroups share each SIMD, so one's softmax phase overlaps the
//      other's matrix phase.  Stage t holds the V rows of blocks 2t, 2t+1 and the K rows of
//      blocks 2t+2, 2t+3 in one of two LDS buffers (separate arrays, so the compiler can see
//      that the direct loads into one never alias reads of the other); the next stage loads
//      during the current step, one barrier per step (between its softmax and matrix phases, whose
//      MFMAs the next stage's loads are issued between).  Step pairs whose next stages are full
//      run with no conditional code; the last steps mask the scores of keys past S.
//   2. drafts: each wave visits only the 32-key tiles holding its own block or an ancestor
//      block (the set bits of the OR of its rows' ancestor masks, lowest first); optional
//      per-draft peer masks add drafts to a draft's visible set (inter-block speculation).
//      Tiles that hold only fully visible blocks need no per-element mask (always the case
//      when L is a multiple of 32 and a wave's rows share a draft).
//   3. with KG key groups of 4 waves (grids of at most one workgroup per CU over longer caches):
//      group kg takes its own range of cache steps and every KG-th draft tile, and the groups'
//      outputs, references and sums are merged through LDS.
//   With drafts_visible = 0 every visible set is empty and phase 2 does nothing: the queries
//   attend to the S cache keys only.  The dual-cache refresh uses this for bidirectional
//   attention over whole sequences (its "cache" is the sequence's own K / V, N = 1 and L = the
//   sequence length, no parent array).
#pragma once

#include "common.hpp"

namespace trajspec {

struct AttnParams {
    const uint16_t* q;
    const uint16_t* kc;
    const uint16_t* vc;
    const uint16_t* kd;
    const uint16_t* vd;
    const int32_t* parent;
    const uint64_t* peers;  // [B,N] extra visible drafts per draft (bit j = draft j), or null
    uint16_t* out;
    int B, N, L, Hq, Hkv, S;
    int group;           // Hq / Hkv
    int rows_per_group;  // group * N * L
    int wg_per_group;    // workgroups per (b, g)
    int num_wg;
    float scale_log2;    // softmax scale * log2(e)
    int drafts_visible;  // 1: each draft sees its root path (+ peers); 0: queries see the cache only
    int warm;            // 16-row kernel: read the cache into L2 ahead of the steps (it comes from HBM)
};

constexpr int kAttnWaves = 4;
// Word 3 of a raw (untyped) buffer descriptor on gfx950: 32-bit data format, no swizzle.
constexpr int kBufferFlags = 0x00020000;
// s_waitcnt immediate (gfx9 encoding) waiting for vector-memory loads only: vmcnt = 0,
// expcnt and lgkmcnt left at their maxima.
constexpr int kWaitVmcnt0 = 0x0F70;
constexpr int kAttnThreads = kAttnWaves * 64;
constexpr int kAttnTile = 64;  // cache keys per LDS tile
// Online softmax: the reference maximum of a query only moves when a new score exceeds it
// by more than this many powers of two, so weights stay below 2^kLazyLog2.
constexpr float kLazyLog2 = 8.0f;

typedef __attribute__((address_space(3))) bf16x4_t lds_bf16x4_t;

// R = query rows per wave (32: v_mfma_f32_32x32x16_bf16; 16: v_mfma_f32_16x16x32_bf16).  Only the
// V tile's chunk swizzle depends on it: it is chosen so that the rows one half-wave reads with a
// transposing load fall into distinct bank groups.
template <int D, int R = 32>
struct AttnGeom {
    static constexpr int kChunks = D / 8;                         // 16-byte chunks per row
    static constexpr int kTileElems = kAttnTile * D;              // one K or V tile
    static constexpr int kStageElems = 2 * kTileElems;            // K tile then V tile
    static constexpr int kRowsPerDma = 512 / D;                   // rows per wave-wide 1 KB load
    static constexpr int kDmaPerWave = (kAttnTile / kAttnWaves) / kRowsPerDma;
    static constexpr int kWaveRegionElems = 2 * 32 * D;           // per-wave draft tile (K, V)
    static constexpr int kDraftDma = 32 / kRowsPerDma;
    static_assert(2 * kWaveRegionElems <= kStageElems, "two draft regions per buffer");

    static __device__ __forceinline__ int k_swz(int r) { return kChunks == 16 ? (r & 15) : ((r >> 1) & 7); }
    static __device__ __forceinline__ int v_rot(int r) {
        if (R == 16) return kChunks == 16 ? ((r & 7) << 1) : (((r >> 1) & 3) << 1);
        return kChunks == 16 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
    }
};

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ bf16x4_t lds_read_tr(const uint16_t* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_t*)(p));
}

__device__ __forceinline__ u32x4_t ldg16(const uint16_t* p) { return *reinterpret_cast<const u32x4_t*>(p); }

__device__ __forceinline__ bf16x8_t lds16(const uint16_t* p) { return *reinterpret_cast<const bf16x8_t*>(p); }

// 16 bytes per lane from global memory straight into LDS; the wave writes the contiguous
// kilobyte starting at lds_row0 (lane i -> bytes 16 i .. 16 i + 15).
__device__ __forceinline__ void dma16(const uint16_t* g, uint16_t* lds_row0) {
    __builtin_amdgcn_global_load_lds((const void*)g, (lds_void_t*)lds_row0, 16, 0, 0);
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)x, off);
        const uint32_t hi = __shfl_xor((uint32_t)(x >> 32), off);
        x |= ((uint64_t)hi << 32) | lo;
    }
    return x;
}

// x combined with the value of lane l^32 (v_permlane32_swap: pure VALU, no LDS round trip).
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x),
                                                    false, false);
    const uint32_t a = r[0], b = r[1];  // copy out: bit_cast of a vector element reads element 0
    return fmaxf(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, x),
                                                    false, false);
    const uint32_t a = r[0], b = r[1];
    return __builtin_bit_cast(float, a) + __builtin_bit_cast(float, b);
}

// Online softmax over 32-key blocks of raw scores (masked keys = -inf).  The lane holds 16
// scores for its query column, lane^32 the other 16.  `m` is the query's reference maximum in
// raw score units and `c` = scale * log2(e), so a weight is exp2(c * (score - m)): one FMA and
// one exp2 per score.  The reference only moves (and O and the running sum are only
// rescaled) when a block maximum exceeds it by more than kLazyLog2 in the log2 domain:
// weights then stay below 2^kLazyLog2, which fp32 accumulators and bf16 weights hold at full
// relative precision, and most blocks skip the rescale.  The decision is per query, the
// branch wave-uniform.
//
// Online-softmax state of one query: reference m (raw score units), -c*m (0 while m = -inf),
// m + thr (the lazy-rescale trigger) and the running sum of weights.  The derived values
// change only when m moves.
struct SoftState {
    float m, neg_mc, mthr, lsum;
};

// block_max_update: fold the block maximum into `m`, rescaling o and lsum when it moves.
// Scores are never NaN (finite inputs, -inf for masked keys), so the NaN-propagating
// maximum (v_maximum3_f32, no operand canonicalisation) is exact here.  `thr` is
// kLazyLog2 / c in raw score units; with m = -inf the test holds exactly when the block has
// a visible key.

// Folds a block maximum mx (already combined with lane^32) into `m`, rescaling o and lsum when
// it moves past the lazy trigger.
template <int D>
__device__ __forceinline__ void fold_max(float mx, float c, float thr, SoftState& st, f32x16_t (&o)[D / 32]) {
    const bool need = mx > st.mthr;
    if (ballot64(need) != 0ull) {
        const float m_new = need ? mx : st.m;
        const float alpha = need ? fast_exp2((st.m - m_new) * c) : 1.0f;  // 0 when m was -inf
        st.lsum *= alpha;
#pragma unroll
        for (int db = 0; db < D / 32; ++db) o[db] *= alpha;
        st.m = m_new;
        st.neg_mc = m_new == kNegInf ? 0.f : -m_new * c;
        st.mthr = m_new + thr;
    }
}

__device__ __forceinline__ float max16(const f32x16_t& s, float mx) {
#pragma unroll
    for (int v = 0; v < 16; v += 2) mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, s[v]), s[v + 1]);
    return mx;
}

template <int D>
__device__ __forceinline__ void block_max_update(const f32x16_t& s, float c, float thr, SoftState& st,
                                                 f32x16_t (&o)[D / 32]) {
    float mx = __builtin_elementwise_maximum(s[0], s[1]);
#pragma unroll
    for (int v = 2; v < 16; v += 2) mx = __builtin_elementwise_maximum(__builtin_elementwise_maximum(mx, s[v]), s[v + 1]);
    fold_max<D>(pair_max(mx), c, thr, st, o);
}

// block_exp: weights of one block against the current reference (neg_mc = -c*m); pf[half]
// receives the bf16 weights of keys 16*half .. +15 in MFMA B-operand order, and lsum grows by
// their fp32 sum.
__device__ __forceinline__ void block_exp(const f32x16_t& s, float c, float neg_mc, float& lsum, bf16x8_t (&pf)[2]) {
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float p = fast_exp2(__builtin_fmaf(s[v], c, neg_mc));
        sum += p;
        pf[v >> 3][v & 7] = (__bf16)p;
    }
    lsum += sum;
}

template <int D>
__device__ __forceinline__ void softmax_update(const f32x16_t& s, float c, float thr, SoftState& st,
                                               f32x16_t (&o)[D / 32], bf16x8_t (&pf)[2]) {
    block_max_update<D>(s, c, thr, st, o);
    block_exp(s, c, st.neg_mc, st.lsum, pf);
}

// Scores of keys key0 .. key0+31 at or beyond S are masked (branch-free select).
__device__ __forceinline__ void mask_tail(f32x16_t& s, int key0, int S, int h) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int key = key0 + 8 * (v >> 2) + 4 * h + (v & 3);
        s[v] = key < S ? s[v] : kNegInf;
    }
}

// S^T of one 32-key block: kbase = K region + block row offset; kq[ks] = this lane's
// fragment offset for k-step ks.
template <int D>
__device__ __forceinline__ f32x16_t qk_block(const uint16_t* kbase, const int (&kq)[D / 16],
                                             const bf16x8_t (&qf)[D / 16]) {
    constexpr int KS = D / 16;
    bf16x8_t ka[KS];
    ka[0] = lds16(kbase + kq[0]);
    ka[1] = lds16(kbase + kq[1]);
    f32x16_t s = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {  // fragment reads two steps ahead, each after an MFMA
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], s, 0, 0, 0);
        if (ks + 2 < KS) ka[ks + 2] = lds16(kbase + kq[ks + 2]);
        __builtin_amdgcn_sched_barrier(0);
    }
    return s;
}

// O^T += V^T P^T for one 32-key block: vbase = V region + block row offset; vq[db] = this
// lane's transposing-read offset for output block db.
template <int D>
__device__ __forceinline__ void pv_block(const uint16_t* vbase, const int (&vq)[D / 32], const bf16x8_t (&pf)[2],
                                         f32x16_t (&o)[D / 32]) {
    constexpr int NDB = D / 32;
    bf16x8_t va[2][NDB];
    auto read_v = [&](int half, int db, bf16x8_t& dst) {
        const bf16x4_t a0 = lds_read_tr(vbase + vq[db] + (16 * half) * D);
        const bf16x4_t a1 = lds_read_tr(vbase + vq[db] + (16 * half + 8) * D);
        dst = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
#pragma unroll
    for (int db = 0; db < NDB; ++db) read_v(0, db, va[0][db]);
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // the second half's reads follow the first half's MFMAs
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[half][db], pf[half], o[db], 0, 0, 0);
            if (half == 0) read_v(1, db, va[1][db]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Per-lane constants of the cache phase.
template <int D>
struct AttnLane {
    int kq[D / 16];   // K fragment offsets (region-relative, elements)
    int vq[D / 32];   // V transposing-read offsets (region-relative, elements)
    int ri;           // row of this lane's chunk within a wave-wide direct load
    int pc;           // LDS chunk slot of this lane within that row
};

// Direct loads of 64 cache rows, keys key0 .. key0+63, into the LDS tile `dst` with the
// chunk swizzle SWZ: wave `wave` (uniform) fills tile rows [16 wave, 16 wave + 16),
// kRowsPerDma rows per load.  The first global row of each load is uniform, so addresses are
// a scalar base plus this lane's 32-bit offset.  RAGGED clamps keys >= S to key S-1 (their
// scores are masked or never computed; the clamped values stay finite); the uniform base row
// is clamped too, so a lane's offset from it is never negative.
template <int D, bool RAGGED, bool IS_V, int R = 32, typename LaneT>
__device__ __forceinline__ void cache_row_dma(__amdgpu_buffer_rsrc_t rs, int kv_stride, int key0, int S, int wave,
                                              const LaneT& ln, uint16_t* dst, int j) {
    using G = AttnGeom<D, R>;
    const int row0 = wave * (kAttnTile / kAttnWaves) + j * G::kRowsPerDma;  // uniform
    const int r = row0 + ln.ri;                                               // tile row
    int base_row = key0 + row0;
    int grow = ln.ri;
    if (RAGGED) {
        base_row = min(base_row, S - 1);
        grow = min(key0 + r, S - 1) - base_row;
    }
    const int swz = IS_V ? G::v_rot(r) : G::k_swz(r);
    const unsigned voff = 2u * (unsigned)(grow * kv_stride + ((ln.pc ^ swz) << 3));  // lane bytes
    const unsigned soff = 2u * (unsigned)(base_row * kv_stride);                     // uniform bytes
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)(dst + row0 * D), 16, voff, soff, 0, 0);
}

template <int D, bool RAGGED, bool IS_V, int R = 32, typename LaneT>
__device__ __forceinline__ void cache_rows_dma(__amdgpu_buffer_rsrc_t rs, int kv_stride, int key0, int S, int wave,
                                               const LaneT& ln, uint16_t* dst) {
#pragma unroll
    for (int j = 0; j < AttnGeom<D, R>::kDmaPerWave; ++j)
        cache_row_dma<D, RAGGED, IS_V, R>(rs, kv_stride, key0, S, wave, ln, dst, j);
}

// Stage t of the cache pipeline holds the V rows of keys 64 t .. 64 t + 63 (blocks 2t, 2t+1) and
// the K rows of keys 64 t + 64 .. 64 t + 127 (blocks 2t+2, 2t+3): the matrix phase of step t
// multiplies the V rows of the blocks whose weights were just computed and the K rows of the
// next two blocks, so one buffer and one barrier per stage suffice.  RAGGED when 64 t + 128 > S.
template <int D, bool RAGGED, int R = 32, typename LaneT>
__device__ __forceinline__ void stage_dma(__amdgpu_buffer_rsrc_t krs, __amdgpu_buffer_rsrc_t vrs, int kv_stride, int t,
                                          int S, int wave, const LaneT& ln, uint16_t* stage) {
    using G = AttnGeom<D, R>;
    cache_rows_dma<D, RAGGED, false, R>(krs, kv_stride, t * kAttnTile + kAttnTile, S, wave, ln, stage);
    cache_rows_dma<D, RAGGED, true, R>(vrs, kv_stride, t * kAttnTile, S, wave, ln, stage + G::kTileElems);
}

// Load i of a full stage t (the K rows' loads, then the V rows').
template <int D, int R = 32, typename LaneT>
__device__ __forceinline__ void stage_dma_one(__amdgpu_buffer_rsrc_t krs, __amdgpu_buffer_rsrc_t vrs, int kv_stride, int t,
                                              int S, int wave, const LaneT& ln, uint16_t* stage, int i) {
    using G = AttnGeom<D, R>;
    if (i < G::kDmaPerWave)
        cache_row_dma<D, false, false, R>(krs, kv_stride, t * kAttnTile + kAttnTile, S, wave, ln, stage, i);
    else
        cache_row_dma<D, false, true, R>(vrs, kv_stride, t * kAttnTile, S, wave, ln, stage + G::kTileElems, i - G::kDmaPerWave);
}

// Softmax phase of a 64-key step: the weights of two blocks (s[0], s[1]) against the query's
// reference; pf[b][half] receives the bf16 weights of block b, keys 16 half .. 16 half + 15, in MFMA
// B-operand order.  A weight exceeds 2^kLazyLog2 exactly when its score passes the lazy trigger, so
// the lane's weight sum of the step is compared with that bound instead of taking the block maximum
// first: only then (or while the reference is still -inf) does the wave take the path that folds the
// true joint maximum in and recomputes.  The reference therefore moves at the same scores as with a
// maximum taken every step (up to the rounding of the two tests at the trigger itself); on every
// workload measured the outputs are the same bits.  Saves 16 three-input maxima, a lane swap and a
// compare per step of each wave.
template <int D>
__device__ __forceinline__ void softmax_phase(const f32x16_t (&s)[2], float c, float thr, SoftState& st,
                                              f32x16_t (&o)[D / 32], bf16x8_t (&pf)[2][2]) {
    float neg_mc = st.neg_mc;
    float sum0 = 0.f, sum1 = 0.f;
    float p0[16], p1[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        p0[v] = fast_exp2(__builtin_fmaf(s[0][v], c, neg_mc));
        p1[v] = fast_exp2(__builtin_fmaf(s[1][v], c, neg_mc));
        sum0 += p0[v];
        sum1 += p1[v];
    }
    const bool big = !(sum0 + sum1 <= (float)(1 << (int)kLazyLog2)) || st.m == kNegInf;
    if (ballot64(big) != 0ull) {
        const float mx = max16(s[1], max16(s[0], kNegInf));
        fold_max<D>(pair_max(mx), c, thr, st, o);
        neg_mc = st.neg_mc;
        sum0 = 0.f;
        sum1 = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            p0[v] = fast_exp2(__builtin_fmaf(s[0][v], c, neg_mc));
            p1[v] = fast_exp2(__builtin_fmaf(s[1][v], c, neg_mc));
            sum0 += p0[v];
            sum1 += p1[v];
        }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        pf[0][v >> 3][v & 7] = (__bf16)p0[v];
        pf[1][v >> 3][v & 7] = (__bf16)p1[v];
    }
    st.lsum += sum0 + sum1;
}

// Scores of two consecutive 32-key blocks whose K rows start at kbase (rows 0..31, 32..63 of a K
// region): two independent MFMA chains, links alternating, fragment reads two links ahead.
template <int D>
__device__ __forceinline__ void qk_pair(const uint16_t* kbase, const AttnLane<D>& ln, const bf16x8_t (&qf)[D / 16],
                                        f32x16_t (&sn)[2]) {
    constexpr int KS = D / 16;
    bf16x8_t ka[KS], kb[KS];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        ka[ks] = lds16(kbase + ln.kq[ks]);
        kb[ks] = lds16(kbase + 32 * D + ln.kq[ks]);
    }
    f32x16_t a = {}, b = {};
    // Each fragment read is issued right after an MFMA, so that it issues while that MFMA
    // executes: a wave issues in order and waits at an MFMA until the previous one has left the
    // pipe, so reads placed after a run of MFMAs would add their issue time to the phase.
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], a, 0, 0, 0);
        if (ks + 2 < KS) ka[ks + 2] = lds16(kbase + ln.kq[ks + 2]);
        __builtin_amdgcn_sched_barrier(0);
        b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[ks], qf[ks], b, 0, 0, 0);
        if (ks + 2 < KS) kb[ks + 2] = lds16(kbase + 32 * D + ln.kq[ks + 2]);
        __builtin_amdgcn_sched_barrier(0);
    }
    sn[0] = a;
    sn[1] = b;
}

// O^T += V^T P^T for two consecutive 32-key blocks whose V rows start at vbase; each (block,
// half) group's transposing reads are issued one group ahead of its MFMAs.
template <int D>
__device__ __forceinline__ void pv_pair(const uint16_t* vbase, const AttnLane<D>& ln, const bf16x8_t (&pf)[2][2],
                                        f32x16_t (&o)[D / 32]) {
    constexpr int NDB = D / 32;
    bf16x8_t va[2][NDB];
    auto read_group = [&](int grp, bf16x8_t (&dst)[NDB]) {
        const uint16_t* base = vbase + (grp >> 1) * 32 * D + (grp & 1) * 16 * D;
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            const bf16x4_t a0 = lds_read_tr(base + ln.vq[db]);
            const bf16x4_t a1 = lds_read_tr(base + ln.vq[db] + 8 * D);
            dst[db] = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    auto read_one = [&](int grp, int db, bf16x8_t& dst) {
        const uint16_t* base = vbase + (grp >> 1) * 32 * D + (grp & 1) * 16 * D;
        const bf16x4_t a0 = lds_read_tr(base + ln.vq[db]);
        const bf16x4_t a1 = lds_read_tr(base + ln.vq[db] + 8 * D);
        dst = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    read_group(0, va[0]);
    // the next group's reads go out one fragment after each MFMA (see qk_pair)
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[grp & 1][db], pf[grp >> 1][grp & 1], o[db], 0, 0, 0);
            if (grp + 1 < 4) read_one(grp + 1, db, va[(grp + 1) & 1][db]);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Matrix phase of a step with both parts: the scores of the next pair from the K rows at kbase
// and O += V P of the current pair from the V rows at vbase.  As in qk_pair / pv_pair every
// fragment read follows an MFMA; the V fragments of the first group ride on the last QK MFMAs,
// which have no K reads left to carry.
template <int D, typename Side>
__device__ __forceinline__ void matrix_pair(const uint16_t* kbase, const uint16_t* vbase, const AttnLane<D>& ln,
                                            const bf16x8_t (&qf)[D / 16], f32x16_t (&sn)[2], const bf16x8_t (&pf)[2][2],
                                            f32x16_t (&o)[D / 32], Side side) {
    constexpr int KS = D / 16;
    constexpr int NDB = D / 32;
    static_assert(2 * 2 >= NDB, "the last two QK steps carry the first V group");
    bf16x8_t ka[KS], kb[KS];
    bf16x8_t va[2][NDB];
    auto read_v = [&](int grp, int db, bf16x8_t& dst) {
        const uint16_t* base = vbase + (grp >> 1) * 32 * D + (grp & 1) * 16 * D;
        const bf16x4_t a0 = lds_read_tr(base + ln.vq[db]);
        const bf16x4_t a1 = lds_read_tr(base + ln.vq[db] + 8 * D);
        dst = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        ka[ks] = lds16(kbase + ln.kq[ks]);
        kb[ks] = lds16(kbase + 32 * D + ln.kq[ks]);
    }
    f32x16_t a = {}, b = {};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], qf[ks], a, 0, 0, 0);
        if (ks + 2 < KS) {
            ka[ks + 2] = lds16(kbase + ln.kq[ks + 2]);
        } else {
            const int db = 2 * (ks + 2 - KS);
            if (db < NDB) read_v(0, db, va[0][db]);
        }
        side(2 * ks);
        __builtin_amdgcn_sched_barrier(0);
        b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kb[ks], qf[ks], b, 0, 0, 0);
        if (ks + 2 < KS) {
            kb[ks + 2] = lds16(kbase + 32 * D + ln.kq[ks + 2]);
        } else {
            const int db = 2 * (ks + 2 - KS) + 1;
            if (db < NDB) read_v(0, db, va[0][db]);
        }
        side(2 * ks + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    sn[0] = a;
    sn[1] = b;
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
            o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[grp & 1][db], pf[grp >> 1][grp & 1], o[db], 0, 0, 0);
            if (grp + 1 < 4) read_v(grp + 1, db, va[(grp + 1) & 1][db]);
            side(2 * KS + grp * NDB + db);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

struct CacheArgs {
    __amdgpu_buffer_rsrc_t krs, vrs;  // this (b, g) cache slice as buffer descriptors
    int kv_stride;
    int S, wave, h;
    float c, thr;
};

// One 64-key step t of the cache phase whose next stage is full (64 t + 192 <= S): the softmax
// phase turns the scores of blocks 2t, 2t+1 into weights; once every wave's loads of stage t have
// landed (wait and barrier), the matrix phase computes the scores of blocks 2t+2, 2t+3, adds the
// weighted V rows of blocks 2t, 2t+1 and issues the loads of stage t+1 between the first half of its MFMAs
// (issued together before the softmax they held it up: the load path takes one per ~16 cycles and CU;
// spread over all the MFMAs the last came too late for a cache in HBM: 16 sequences of 64 drafts x 32 over
// 4096 keys 1969 us, 1932 so, 64 drafts of 4 sequences over 2048 keys 278 -> 275, of 11 x 8 over 3000 179 -> 173).
// Two waves share each SIMD: one's softmax phase runs on the vector ALU while the other's matrix
// phase runs on the matrix core.
template <int D>
__device__ __forceinline__ void full_step(int t, const CacheArgs& a, const AttnLane<D>& ln, const uint16_t* cur,
                                          uint16_t* nxt, const bf16x8_t (&qf)[D / 16], f32x16_t (&s)[2], SoftState& st,
                                          f32x16_t (&o)[D / 32]) {
    using G = AttnGeom<D>;
    constexpr int NM = D / 16 + 2 * (D / 32), NL = 2 * G::kDmaPerWave;  // MFMAs that loads follow, loads
    bf16x8_t pf[2][2];
    softmax_phase<D>(s, a.c, a.thr, st, o, pf);
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    // the matrix phase issues at a raised wave priority: when the other wave on the SIMD is in
    // its softmax phase, the arbiter then keeps the matrix core fed first (-6% on 8b-batched)
    __builtin_amdgcn_s_setprio(1);
    matrix_pair<D>(cur, cur + G::kTileElems, ln, qf, s, pf, o, [&](int i) {
        if (i < NM && (i + 1) * NL / NM > i * NL / NM)
            stage_dma_one<D>(a.krs, a.vrs, a.kv_stride, t + 1, a.S, a.wave, ln, nxt, i * NL / NM);
    });
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
}

// Ascending walk over the 32-key draft tiles that hold a block of `todo` (a wave-uniform set of
// drafts): block j covers tiles (j L) / 32 .. (j L + L - 1) / 32, and a tile that an earlier
// (lower) block already covered is not visited again.  cur .. hi are the current block's
// remaining tiles; next() returns the next tile, or -1 once every block is done.
struct TileWalk {
    uint64_t todo;
    int cur, hi;
    __device__ __forceinline__ int next(int L) {
        while (cur > hi) {
            if (todo == 0ull) return -1;
            const int jb = __builtin_ctzll(todo);
            todo &= todo - 1ull;
            cur = max((jb * L) >> 5, hi + 1);  // blocks ascend, so hi + 1 is the first tile not yet visited
            hi = (jb * L + L - 1) >> 5;
        }
        return cur++;
    }
};

// A wave-uniform 64-bit value moved to scalar registers (the compiler cannot see that the result of
// a lane-exchange reduction is uniform).
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Orders a wave's LDS accesses around direct loads into its own region (no other wave touches it).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Per-wave constants of the draft phase.
struct DraftArgs {
    const uint16_t* kd;  // this K/V head's column of the packed draft keys / values
    const uint16_t* vd;
    int64_t seq_row0;    // b * N * L: first packed draft row of the sequence
    int NL, N, L, kv_stride;
    int wri, wpc;        // row and chunk slot of this lane within a wave-wide direct load
    uint64_t anc;        // this lane's visible drafts (0 for rows past the workgroup's share)
    bool row_valid;
    int h;
};

template <int D>
__device__ __forceinline__ DraftArgs draft_args(const AttnParams& P, int b, int g, int lane, uint64_t my_anc,
                                                bool row_valid, int h) {
    using G = AttnGeom<D>;
    DraftArgs a;
    a.kd = P.kd + (int64_t)g * D;
    a.vd = P.vd + (int64_t)g * D;
    a.NL = P.N * P.L;
    a.seq_row0 = (int64_t)b * a.NL;
    a.N = P.N;
    a.L = P.L;
    a.kv_stride = P.Hkv * D;
    a.wri = lane / G::kChunks;
    a.wpc = lane % G::kChunks;
    a.anc = my_anc;
    a.row_valid = row_valid;
    a.h = h;
    return a;
}

// Direct loads of the 32 draft keys k0 .. k0+31 into a wave's tile regions kw (K rows) and vw
// (V rows), with the cache tiles' swizzles.  Rows past the packed drafts read the last draft key;
// base and lane row are both clamped so the lane offset is never negative (those keys are masked).
template <int D, int R = 32>
__device__ __forceinline__ void draft_tile_dma(const DraftArgs& a, int k0, uint16_t* kw, uint16_t* vw) {
    using G = AttnGeom<D, R>;
#pragma unroll
    for (int j = 0; j < G::kDraftDma; ++j) {
        const int row0 = j * G::kRowsPerDma;
        const int r = row0 + a.wri;
        const int base_row = min(k0 + row0, a.NL - 1);
        const int grow = min(k0 + r, a.NL - 1) - base_row;
        const int64_t rowbase = (a.seq_row0 + base_row) * a.kv_stride;  // uniform
        const unsigned ok = (unsigned)(grow * a.kv_stride + ((a.wpc ^ G::k_swz(r)) << 3));
        const unsigned ov = (unsigned)(grow * a.kv_stride + ((a.wpc ^ G::v_rot(r)) << 3));
        dma16(a.kd + rowbase + ok, kw + row0 * D);
        dma16(a.vd + rowbase + ov, vw + row0 * D);
    }
}

// Scores, weights and O += V P of the draft tile k0 .. k0+31 held in the wave's regions kw, vw.
template <int D>
__device__ __forceinline__ void draft_tile(const DraftArgs& a, int k0, const uint16_t* kw, const uint16_t* vw,
                                           const AttnLane<D>& ln,
                                           const bf16x8_t (&qf)[D / 16], SoftState& st, f32x16_t (&o)[D / 32],
                                           float c, float thr) {
    const int jlo = k0 / a.L;
    const int jhi = min(a.N - 1, (k0 + 31) / a.L);
    const uint64_t T = (jhi - jlo == 63) ? ~0ull : (((1ull << (jhi - jlo + 1)) - 1) << jlo);
    const bool lane_full = !a.row_valid || ((a.anc & T) == T);
    const bool all_full = ballot64_all(lane_full);
    const bool full = (k0 + 32 <= a.NL) & all_full;
    f32x16_t s = qk_block<D>(kw, ln.kq, qf);
    if (!full) {
        // branch-free per-element visibility (key beyond the packed drafts, or a block that is
        // not on this row's root path)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int key = k0 + 8 * (v >> 2) + 4 * a.h + (v & 3);
            const int blk = min(key, a.NL - 1) / a.L;
            const bool vis = (key < a.NL) & (((a.anc >> blk) & 1ull) != 0ull);
            s[v] = vis ? s[v] : kNegInf;
        }
    }
    bf16x8_t pf[2];
    softmax_update<D>(s, c, thr, st, o, pf);
    pv_block<D>(vw, ln.vq, pf, o);
}

template <int D, int KG>
__global__ __launch_bounds__(kAttnThreads* KG, 2 / KG) void verify_attn_kernel(AttnParams P) {
    using G = AttnGeom<D>;
    __shared__ __attribute__((aligned(1024))) uint16_t buf0_all[KG * G::kStageElems];
    __shared__ __attribute__((aligned(1024))) uint16_t buf1_all[KG * G::kStageElems];
    __shared__ uint64_t anc[64];
    __shared__ float merge_m[KG > 1 ? (KG - 1) * kAttnThreads : 1], merge_l[KG > 1 ? (KG - 1) * kAttnThreads : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform per wave
    const int wave = wave_all % kAttnWaves, kg = wave_all / kAttnWaves;  // wave within its key group
    uint16_t* buf0 = buf0_all + kg * G::kStageElems;
    uint16_t* buf1 = buf1_all + kg * G::kStageElems;
    const int h = lane >> 5;

    const int lid = xcd_logical_id(blockIdx.x, P.num_wg);
    const int wg_in_group = lid % P.wg_per_group;
    const int bg = lid / P.wg_per_group;
    const int g = bg % P.Hkv;
    const int b = bg / P.Hkv;
    const int N = P.N, L = P.L;
    const float c = P.scale_log2;
    const float thr = kLazyLog2 / c;  // lazy-rescale margin in raw score units

    // The parent array (ancestor walk below) is loaded first: the walk then waits for this
    // load only, not for the Q, K and stage loads issued after it.
    const int pj = (P.parent != nullptr && wave_all == 0 && lane < N) ? P.parent[(int64_t)b * N + lane] : -1;
    const uint64_t peer_bits = (P.peers != nullptr && wave_all == 0 && lane < N) ? P.peers[(int64_t)b * N + lane] : 0ull;

    // This lane's query row (lanes l and l^32 share a row).
    const int row = (wg_in_group * kAttnWaves + wave) * 32 + (lane & 31);
    const bool row_valid = row < P.rows_per_group;
    const int NL = N * L;
    // query row -> (head in group, draft, position) and the element offset of its q / out row
    auto row_offset = [&](int& nd_out) -> int64_t {
        const int hg = row / NL;
        const int rem = row - hg * NL;
        nd_out = rem / L;
        const int p = rem - nd_out * L;
        return ((((int64_t)b * N + nd_out) * L + p) * P.Hq + (g * P.group + hg)) * D;
    };
    int nd_q = 0;
    const int64_t row_off_q = row_valid ? row_offset(nd_q) : 0;
    bf16x8_t qf[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        if (row_valid) {
            qf[ks] = __builtin_bit_cast(bf16x8_t, ldg16(P.q + row_off_q + ks * 16 + h * 8));
        } else {
            qf[ks] = bf16x8_t{};
        }
    }
    // The Q loads are retired by the prologue's wait below (together with block 0 and stage 0),
    // so no use of Q inside the tile loop waits on a later stage's loads.

    const int kv_stride = P.Hkv * D;  // elements between consecutive keys
    AttnLane<D> ln;
    {
        const int r = lane & 31;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) ln.kq[ks] = r * D + (((2 * ks + h) ^ G::k_swz(r)) << 3);
        const int i = lane & 15;
        const int dsub = (lane >> 4) & 1;
        const int vr = 4 * h + (i >> 2);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
            const int chunk = db * 4 + 2 * dsub + ((i & 3) >> 1);
            ln.vq[db] = vr * D + ((chunk ^ G::v_rot(vr)) << 3) + (i & 1) * 4;
        }
        ln.ri = lane / G::kChunks;
        ln.pc = lane % G::kChunks;
    }

    f32x16_t o[D / 32];
#pragma unroll
    for (int db = 0; db < D / 32; ++db) o[db] = f32x16_t{};
    SoftState st = {kNegInf, 0.f, kNegInf, 0.f};

    // ---------------- phase 1: cache keys ----------------
    // this group's keys: steps [kg steps_max, (kg + 1) steps_max) of the cache
    const int steps_max = ((P.S + kAttnTile - 1) / kAttnTile + KG - 1) / KG;
    const int key_first = min(kg * steps_max * kAttnTile, P.S);
    const int S = min(steps_max * kAttnTile, P.S - key_first);
    CacheArgs ca;
    {
        // descriptors over this (b, g) slice to the end of the tensor (the host guarantees one
        // sequence's cache spans less than 2^31 bytes, so row offsets fit the 32-bit soffset)
        const int64_t first = (((int64_t)b * P.S + key_first) * P.Hkv + g) * D;
        const uint16_t* kc_base = P.kc + first;
        const uint16_t* vc_base = P.vc + first;
        const int64_t total = (int64_t)P.B * P.S * P.Hkv * D * 2;
        const int64_t start = first * 2;
        const int64_t rem = total - start;
        const int nrec = rem > 0x7FFFFFFF ? 0x7FFFFFFF : rem < 0 ? 0 : (int)rem;
        ca.krs = __builtin_amdgcn_make_buffer_rsrc((void*)kc_base, (short)0, nrec, kBufferFlags);
        ca.vrs = __builtin_amdgcn_make_buffer_rsrc((void*)vc_base, (short)0, nrec, kBufferFlags);
    }
    ca.kv_stride = kv_stride;
    ca.S = S;
    ca.wave = wave;
    ca.h = h;
    ca.c = c;
    ca.thr = thr;

    const int nb = (S + 31) / 32;    // 32-key blocks
    const int nst = (nb + 1) / 2;    // 64-key steps, one stage each
    f32x16_t s[2] = {{}, {}};        // scores of the step's two blocks
    if (nb > 0) {
        // the K rows of keys 0..63 go to buf1's K region (free until stage 1), stage 0 to buf0
        if (64 <= S) {
            cache_rows_dma<D, false, false>(ca.krs, kv_stride, 0, S, wave, ln, buf1);
        } else {
            cache_rows_dma<D, true, false>(ca.krs, kv_stride, 0, S, wave, ln, buf1);
        }
        if (128 <= S) {
            stage_dma<D, false>(ca.krs, ca.vrs, kv_stride, 0, S, wave, ln, buf0);
        } else {
            stage_dma<D, true>(ca.krs, ca.vrs, kv_stride, 0, S, wave, ln, buf0);
        }
    }
    // Ancestor masks (bit j of anc[n] set when draft j is n itself or on n's root path).  Wave 0
    // holds the sequence's parent array (N <= 64 = one value per lane) and every lane walks
    // its own draft's chain through lane shuffles, so the walk costs no dependent global loads.
    if (wave_all == 0) {
        uint64_t msk = 1ull << lane;
        int j = pj, prev = lane;
        bool live = lane < N;
        while (true) {  // every step moves prev strictly down, so at most N steps
            const bool step = live && j != -1;
            const bool bad = step && (j < -1 || j >= prev);  // not topological: report, stop here
            if (bad) flag_device_status(1);
            const bool go = step && !bad;
            if (ballot64(go) == 0ull) break;
            if (go) {
                msk |= 1ull << j;
                prev = j;
            }
            const int nj = __shfl(pj, go ? j : 0);
            j = go ? nj : -1;
            live = go;
        }
        // drafts made visible beyond the root path (the joint trees of inter-block
        // speculation), restricted to the N drafts of the sequence
        const uint64_t in_range = N == 64 ? ~0ull : ((1ull << N) - 1ull);
        if (lane < N) anc[lane] = P.drafts_visible ? (msk | (peer_bits & in_range)) : 0ull;
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __syncthreads();
    if (nb > 0) {
        qk_pair<D>(buf1, ln, qf, s);
        if (S < 64) {
            mask_tail(s[0], 0, S, h);
            mask_tail(s[1], 32, S, h);
        }
    }
    int t = 0;
    // Step pairs whose next stages are full: buffers known at compile time, no conditional code.
    for (; 64 * t + 256 <= S; t += 2) {
        full_step<D>(t, ca, ln, buf0, buf1, qf, s, st, o);
        full_step<D>(t + 1, ca, ln, buf1, buf0, qf, s, st, o);
    }
    // Remaining steps (at most three): clamped loads, masked scores of blocks reaching past S,
    // no scores after the last block.  Blocks past S get weight 0 (their scores are masked and
    // their clamped K / V rows are finite).
    for (; t < nst; ++t) {
        uint16_t* cur = (t & 1) ? buf1 : buf0;
        uint16_t* nxt = (t & 1) ? buf0 : buf1;
        bf16x8_t pf[2][2];
        softmax_phase<D>(s, c, thr, st, o, pf);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < nst) {
            if (64 * t + 192 <= S) {
                stage_dma<D, false>(ca.krs, ca.vrs, kv_stride, t + 1, S, wave, ln, nxt);
            } else {
                stage_dma<D, true>(ca.krs, ca.vrs, kv_stride, t + 1, S, wave, ln, nxt);
            }
        }
        if (2 * t + 2 < nb) {
            qk_pair<D>(cur, ln, qf, s);
            if (64 * t + 128 > S) {
                mask_tail(s[0], 64 * t + 64, S, h);
                mask_tail(s[1], 64 * t + 96, S, h);
            }
        }
        pv_pair<D>(cur + G::kTileElems, ln, pf, o);
    }
    for (; t < steps_max; ++t) __syncthreads();  // a group with fewer steps meets the others' barriers
    __syncthreads();  // the stage buffers are free for the waves' draft tiles; the ancestor masks visible

    // ---------------- phase 2: draft blocks on the root path ----------------
    int nd = 0;
    if (row_valid) (void)row_offset(nd);
    const uint64_t my_anc = row_valid ? anc[nd] : 0ull;
    const DraftArgs da = draft_args<D>(P, b, g, lane, my_anc, row_valid, h);
    // Visit the 32-key tiles that hold a block of any row's root path, in ascending order; each
    // tile is loaded into the wave's region, then multiplied.
    uint16_t* kw = (wave < 2 ? buf0 : buf1) + (wave & 1) * G::kWaveRegionElems;
    TileWalk walk{uniform64(wave_or64(my_anc)), 0, -1};
    int turn = 0;
    for (int tt = walk.next(L); tt >= 0; tt = walk.next(L)) {
        if (KG > 1 && turn++ % KG != kg) continue;  // uniform: the groups take the tiles in turn
        wave_lds_sync();
        draft_tile_dma<D>(da, tt * 32, kw, kw + 32 * D);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        wave_lds_sync();
        draft_tile<D>(da, tt * 32, kw, kw + 32 * D, ln, qf, st, o, c, thr);
    }

    // ---------------- merge the key groups ----------------
    // wave w of every group holds the same rows in the same lanes; a wave's output goes to its own
    // draft tile region (64 lanes x D / 2 floats fill it)
    if (KG > 1) {
        constexpr int NF = D / 2;  // output values per lane
        static_assert(64 * NF * 4 <= G::kWaveRegionElems * 2, "a wave's output fits its draft region");
        wave_lds_sync();
        if (kg > 0) {
            float* f = reinterpret_cast<float*>(kw) + lane;
#pragma unroll
            for (int i = 0; i < NF; ++i) f[64 * i] = o[i >> 4][i & 15];
            merge_m[tid - kAttnThreads] = st.m;
            merge_l[tid - kAttnThreads] = st.lsum;
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int og = 1; og < KG; ++og) {
            const float* f = reinterpret_cast<const float*>(kw + og * G::kStageElems) + lane;
            const float m2 = merge_m[tid + (og - 1) * kAttnThreads], l2 = merge_l[tid + (og - 1) * kAttnThreads];
            const float m = fmaxf(st.m, m2);
            const float a1 = st.m == kNegInf ? 0.f : fast_exp2((st.m - m) * c);
            const float a2 = m2 == kNegInf ? 0.f : fast_exp2((m2 - m) * c);
#pragma unroll
            for (int i = 0; i < NF; ++i) o[i >> 4][i & 15] = o[i >> 4][i & 15] * a1 + f[64 * i] * a2;
            st.lsum = st.lsum * a1 + l2 * a2;
            st.m = m;
        }
    }

    // ---------------- epilogue ----------------
    const float l = pair_sum(st.lsum);
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    if (row_valid) {
        int nd_o = 0;
        const int64_t row_off = row_offset(nd_o);
#pragma unroll
        for (int db = 0; db < D / 32; ++db) {
#pragma unroll
            for (int vg = 0; vg < 4; ++vg) {
                const int d = db * 32 + 8 * vg + 4 * h;
                u32x2_t w;
                const __bf16 e0 = (__bf16)(o[db][4 * vg + 0] * inv);
                const __bf16 e1 = (__bf16)(o[db][4 * vg + 1] * inv);
                const __bf16 e2 = (__bf16)(o[db][4 * vg + 2] * inv);
                const __bf16 e3 = (__bf16)(o[db][4 * vg + 3] * inv);
                w[0] = (uint32_t)__builtin_bit_cast(uint16_t, e0) | ((uint32_t)__builtin_bit_cast(uint16_t, e1) << 16);
                w[1] = (uint32_t)__builtin_bit_cast(uint16_t, e2) | ((uint32_t)__builtin_bit_cast(uint16_t, e3) << 16);
                *reinterpret_cast<u32x2_t*>(P.out + row_off + d) = w;
            }
        }
    }
}

}  // namespace trajspec
