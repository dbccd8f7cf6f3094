// Dense bf16 projection GEMM of the verification layer: D[M,N] = A[M,K] W[K,N] (+ D), all
// row-major bf16, fp32 accumulation on v_mfma_f32_32x32x16_bf16, one bf16 rounding (nearest
// even) of each result.  A holds the packed draft tokens (M = B N L rows), W a weight matrix.
//
// Tilings: gemm_ring_kernel (64 x 64 .. 256 x 128 tiles) and gemm_tile256_kernel (256 x 256), chosen
// by the host from the sizes.
//
// Fragments: the MFMA takes 8 k-values per lane; lane half h = lane / 32 holds k = 8h .. 8h+7
// of each 16-wide k slice, for row (A) or column (W) lane % 32.  A is k-contiguous, so an A
// fragment is one 16-byte LDS read.  W is n-contiguous: a W fragment is two transposing
// reads (ds_read_b64_tr_b16) of slice rows 8h .. 8h+3 and 8h+4 .. 8h+7; in each group of 16
// lanes, lane i addresses 4 columns of row (i / 4) and receives column i of the 4 rows.
//
// LDS layouts (16-byte chunks permuted per row; conflict-free for each reader and writer):
//   A stage [rows][64]: chunk c of row r at c ^ ((r >> 1) & 7)   (16 rows of one chunk: 64 banks)
//   W stage [rows][cols]: chunk c of row r at c ^ ((r & 3) << 2) for multiples of 128 columns
//                       (4 rows x 64 bytes: 64 banks; the permutation stays within 16 chunks)
//
// Loads: operand tiles go global -> LDS directly (buffer_load_dwordx4 ... lds, 1 KB per
// wave-wide load, each lane fetching the chunk that the row permutation puts in its slot).
// Buffer descriptors bound A to the tile's rows and W to the rows below K; chunks past K or N
// get an offset beyond every descriptor's size.  Out-of-range buffer loads return zeros, so
// the edges contribute nothing.  N and K are multiples of 8, M is arbitrary.
//
// Tile order: consecutive logical tiles run on one XCD (one L2) at about the same time; they
// are grouped kGemmGroupM row tiles at a time, so both A and W tiles are reused from L2 (a plain
// row- or column-major order re-reads one operand from HBM once per tile of the other).
//
// Epilogue: the tile's results go through LDS (bf16, row-major) so that global reads of the old
// D (accumulate) and the stores are whole 16-byte chunks, predicated on row < M and
// column < N; with accumulate each result is added to the old value in fp32 and rounded once;
// with SwiGLU the tile holds gate columns and the up columns beside them and silu(gate) * up is stored.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace trajspec {

constexpr int kGemmBK = 64;
constexpr int kGemmGroupM = 8;  // row tiles per ordering group

typedef __attribute__((address_space(3))) bf16x4_t gemm_lds_bf16x4_t;
typedef __attribute__((address_space(3))) void gemm_lds_void_t;

struct GemmParams {
    const uint16_t* A;  // [M, K]
    const uint16_t* W;  // [K, N]
    uint16_t* D;        // [M, N]
    int M, N, K;
    int tiles_m;        // row tiles
    int tiles_n;        // column tiles; the grid holds tiles_m * tiles_n workgroups (x)
    float* partial;     // split-K: [splits][M][N] fp32 partial products (grid y = split)
    int k_split;        // split-K: k per split, a multiple of 64
};

// Limits of the tilings' 32-bit buffer offsets.
constexpr int64_t kGemmMaxK = 1 << 22;              // 256 rows of A below 2^31 bytes
constexpr int64_t kGemmMaxN = 1 << 24;              // 64 rows of W below 2^31 bytes
constexpr int64_t kGemmMaxRecords = 0xFFFFFF00u;    // descriptor sizes stay below the outside offset
constexpr unsigned kGemmOutside = 0xFFFFFFF0u;      // a buffer offset past every descriptor's size
// Word 3 of a raw buffer descriptor on gfx950: 32-bit data format, no swizzle.
constexpr int kGemmBufferFlags = 0x00020000;

// s_waitcnt immediate (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt and lgkmcnt at
// their maxima) waiting until at most n vector-memory loads are outstanding.
constexpr int wait_vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Logical tile of workgroup `bid` in the grouped, XCD-aware order.
__device__ __forceinline__ void gemm_tile_origin(const GemmParams& P, int bm, int bn, int& m0, int& n0) {
    const int tile = xcd_logical_id(blockIdx.x, gridDim.x);
    const int per_group = kGemmGroupM * P.tiles_n;
    const int group = tile / per_group;
    const int first_m = group * kGemmGroupM;
    const int group_m = min(P.tiles_m - first_m, kGemmGroupM);
    const int in_group = tile - group * per_group;
    m0 = (first_m + in_group % group_m) * bm;
    n0 = (in_group / group_m) * bn;
}

__device__ __forceinline__ int gemm_a_slot(int r, int c) { return r * kGemmBK + ((c ^ ((r >> 1) & 7)) << 3); }

// Raw buffer descriptor (gfx950): base address, no stride, num_records bytes, word 3 flags.
typedef int32_t gemm_i32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ gemm_i32x4_t gemm_descriptor(const void* base, unsigned num_records) {
    const uint64_t a = reinterpret_cast<uint64_t>(base);
    return gemm_i32x4_t{(int32_t)(uint32_t)a, (int32_t)((a >> 32) & 0xFFFFu), (int32_t)num_records, kGemmBufferFlags};
}

// One wave-wide 16-byte-per-lane load from a buffer straight into LDS (lane i -> bytes 16 i ..
// 16 i + 15 after the uniform LDS byte offset `lds`).  Issued through asm so that the compiler
// does not track it: with loads into several ring buffers outstanding, its own wait insertion
// cannot tell which buffer they write and would wait for all of them before every LDS read.
// Completion is the caller's explicit s_waitcnt vmcnt; a compiler-tracked load issued earlier
// only sees stricter waits because of these (loads complete in order).
// M0 (the LDS destination of the load) is a register the compiler reserves: the statement
// saves it in a scratch SGPR and restores it after the load, so no code around it sees a
// changed M0.  On gfx9 an SALU write of M0 needs one wait state before an LDS-DMA load reads
// it (the compiler's hazard recognizer does not look inside asm), hence the s_nop.
// NT: non-temporal, for an operand that few other workgroups read, and at about the same time.
template <bool NT>
__device__ __forceinline__ void gemm_dma16(const gemm_i32x4_t& rsrc, unsigned voffset, unsigned lds) {
    unsigned saved;
    if (NT)
        asm volatile(
            "s_mov_b32 %0, m0\n\t"
            "s_mov_b32 m0, %1\n\t"
            "s_nop 0\n\t"
            "buffer_load_dwordx4 %2, %3, 0 offen nt lds\n\t"
            "s_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds), "v"(voffset), "s"(rsrc)
            : "memory");
    else
        asm volatile(
            "s_mov_b32 %0, m0\n\t"
            "s_mov_b32 m0, %1\n\t"
            "s_nop 0\n\t"
            "buffer_load_dwordx4 %2, %3, 0 offen lds\n\t"
            "s_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds), "v"(voffset), "s"(rsrc)
            : "memory");
}

// Workgroup barrier for a stage ring.  __syncthreads() carries a workgroup release fence,
// which waits for every outstanding direct-to-LDS load and would leave one stage in flight.
// Here each wave first waits (s_waitcnt) for exactly the loads of the stage the next step
// reads; the bare s_barrier then makes them visible to every wave (LDS has no caches), and
// the empty asm statements with a memory clobber keep the compiler from moving LDS reads or
// writes across it.  Reads of a stage are consumed by MFMAs before the barrier, so they are
// complete before any wave refills that buffer.
__device__ __forceinline__ void ring_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---------------------------------------------------------------- tiles below 256 x 256
// One kernel body for the smaller grids: BM x BN tiles by WM x WN waves, K in steps of 64
// through a ring of S stages (A [BM][64], W [64][BN]).
//   * A step's 4 slices of 16 k run in clusters of KC slices.  While a cluster multiplies, the
//     fragments of the next cluster are read from LDS, one after each MFMA, and the direct loads
//     are issued between the MFMAs: the load path takes one wave-wide load per ~16 cycles and CU,
//     so a step's loads issued together would hold up every wave's first MFMA.
//   * Step t's last cluster reads the first fragments of stage t + 1, so the workgroup meets before
//     it: there every wave has read all of stage t (its slot is free for stage t + S) and has
//     waited for its loads of stage t + 1; S - 2 more stages stay in flight.
//   * Loads past the k range return zeros into slots that are not multiplied again, so the loop
//     needs no special last steps.
enum GemmEpilogue { kEpiStore, kEpiAccumulate, kEpiPartial, kEpiSwiglu };

// silu(gate) * up of 8 bf16 pairs, fp32 arithmetic, rounded to bf16.
__device__ __forceinline__ u32x4_t swiglu8(const u32x4_t& g, const u32x4_t& u) {
    u32x4_t o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float g0 = bf16_lo(g[e]), g1 = bf16_hi(g[e]);
        const float a = g0 / (1.0f + __expf(-g0)) * bf16_lo(u[e]);
        const float c = g1 / (1.0f + __expf(-g1)) * bf16_hi(u[e]);
        o[e] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)a) | ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)c) << 16);
    }
    return o;
}

// Results of a BM x BN tile through LDS (free, [BM][BN] bf16 row-major): the old D tile is staged
// first when accumulating, each lane adds its fp32 results to it and rounds once; whole 16-byte
// chunks go to memory.  acc[am][bn][e] is row 8 (e / 4) + 4 (lane / 32) + e % 4, column lane % 32
// of its 32 x 32 block.  SwiGLU: the staged columns are BN / 2 gate values, then their up values
// (both rounded to bf16); silu(gate) * up goes to D [M, N / 2].
template <int BM, int BN, int WM, int WN, int EPI, int MB, int NB>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& P, f32x16_t (&acc)[MB][NB], uint16_t* lds, int m0, int n0) {
    constexpr int THREADS = WM * WN * 64, CPR = BN / 8;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN, r32 = lane & 31, h = lane >> 5;
    const int M = P.M, N = P.N;
    static_assert(BM * CPR % THREADS == 0, "whole chunks per thread");
    if (EPI == kEpiAccumulate) {
#pragma unroll
        for (int i = 0; i < BM * CPR / THREADS; ++i) {
            const int q = tid + i * THREADS, r = q / CPR, c = q - r * CPR;
            u32x4_t v = u32x4_t{0, 0, 0, 0};
            if (m0 + r < M && n0 + 8 * c < N) v = *reinterpret_cast<const u32x4_t*>(P.D + (int64_t)(m0 + r) * N + n0 + 8 * c);
            *reinterpret_cast<u32x4_t*>(lds + 8 * q) = v;
        }
        __syncthreads();
    }
#pragma unroll
    for (int am = 0; am < MB; ++am) {
#pragma unroll
        for (int bn = 0; bn < NB; ++bn) {
            const int c = wn * (BN / WN) + bn * 32 + r32;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                uint16_t* p = lds + (wm * (BM / WM) + am * 32 + 8 * (e >> 2) + 4 * h + (e & 3)) * BN + c;
                float v = acc[am][bn][e];
                if (EPI == kEpiAccumulate) v += bf16_bits_to_float(*p);
                *p = __builtin_bit_cast(uint16_t, (__bf16)v);  // round to nearest even
            }
        }
    }
    __syncthreads();
    if (EPI == kEpiSwiglu) {
        constexpr int HC = CPR / 2;
        const int I = N / 2;
        static_assert(BM * HC % THREADS == 0, "whole chunks per thread");
#pragma unroll
        for (int i = 0; i < BM * HC / THREADS; ++i) {
            const int q = tid + i * THREADS, r = q / HC, c = q - r * HC;
            if (m0 + r < M && n0 + 8 * c < I)
                *reinterpret_cast<u32x4_t*>(P.D + (int64_t)(m0 + r) * I + n0 + 8 * c) =
                    swiglu8(*reinterpret_cast<const u32x4_t*>(lds + r * BN + 8 * c),
                            *reinterpret_cast<const u32x4_t*>(lds + r * BN + BN / 2 + 8 * c));
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < BM * CPR / THREADS; ++i) {
        const int q = tid + i * THREADS, r = q / CPR, c = q - r * CPR;
        if (m0 + r < M && n0 + 8 * c < N)
            *reinterpret_cast<u32x4_t*>(P.D + (int64_t)(m0 + r) * N + n0 + 8 * c) = *reinterpret_cast<const u32x4_t*>(lds + 8 * q);
    }
}

template <int BM, int BN, int WM, int WN, int S, int KC, bool NT, int EPI>
__global__ __launch_bounds__(WM* WN * 64, 1) void gemm_ring_kernel(GemmParams P) {
    constexpr int NW = WM * WN;
    constexpr int MB = BM / WM / 32, NB = BN / WN / 32;  // MFMA blocks per wave
    constexpr int NC = 4 / KC;                           // clusters per step
    constexpr int CPR = BN / 8;                          // 16-byte chunks per W row
    constexpr int AE = BM * kGemmBK, SE = AE + kGemmBK * BN;  // elements: A part, stage
    constexpr int LA = BM / 8 / NW, LW = BN / 8 / NW, LS = LA + LW;  // wave-wide loads per wave and stage
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0, "whole wave loads");
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "whole MFMA blocks");
    static_assert((S - 2) * LS < 64, "vmcnt has 6 bits");
    static_assert(S * SE * 2 <= 160 * 1024 && BM * BN <= S * SE, "LDS");
    // XOR on the chunk index of W row r: the 4 rows x 64 bytes that half a wave reads with one
    // transposing load cover all 64 banks (rows of an odd multiple of 64 bytes need none)
    constexpr int QS = BN / 32 % 4;
    auto wswz = [](int r) { return QS == 0 ? (r & 3) << 2 : QS == 2 ? ((r >> 1) & 1) << 2 : 0; };

    __shared__ __attribute__((aligned(1024))) uint16_t lds[S * SE];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int m0, n0;
    gemm_tile_origin(P, BM, EPI == kEpiSwiglu ? BN / 2 : BN, m0, n0);
    const int M = P.M, N = P.N, K = P.K;
    const int kb = EPI == kEpiPartial ? (int)blockIdx.y * P.k_split : 0;  // this workgroup's k range
    const int ke = EPI == kEpiPartial ? min(K, kb + P.k_split) : K;
    const unsigned lds0 = (unsigned)(size_t)((gemm_lds_void_t*)lds);

    const int a_rows = min(M - m0, BM);
    unsigned a_off[LA], w_off[LW];
    int a_kc[LA];
#pragma unroll
    for (int j = 0; j < LA; ++j) {  // 8 rows per load; slot chunk lane & 7 of a row holds chunk (lane & 7) ^ ((row >> 1) & 7)
        const int r = 8 * (wave * LA + j) + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        a_kc[j] = 8 * c;
        a_off[j] = (unsigned)r * (unsigned)K * 2u + 16u * (unsigned)c;
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
        const int q = (wave * LW + j) * 64 + lane;
        const int r = q / CPR;
        const int c = (q - r * CPR) ^ wswz(r);
        // SwiGLU: the tile's columns are BN / 2 gate columns, then the up columns beside them
        const bool up = EPI == kEpiSwiglu && c >= CPR / 2;
        const int col = up ? 8 * c - BN / 2 : 8 * c;
        const bool in = n0 + col < (EPI == kEpiSwiglu ? N / 2 : N);
        w_off[j] = in ? ((unsigned)r * (unsigned)N + (unsigned)(up ? col + N / 2 : col)) * 2u : kGemmOutside;
    }
    const int nk = (ke - kb + kGemmBK - 1) / kGemmBK;
    // the next stage to load
    const uint16_t* a_ptr = P.A + (int64_t)m0 * K + kb;
    const uint16_t* w_ptr = P.W + (int64_t)kb * N + n0;
    int64_t w_rem = ((int64_t)(ke - kb) * N - n0) * 2;
    int l_k = kb;
    unsigned l_dst = lds0;  // of its LDS slot
    gemm_i32x4_t ars, wrs;
    auto begin_stage = [&]() {
        if (ke - l_k < kGemmBK) {  // the last, ragged stage: chunks past ke go outside
#pragma unroll
            for (int j = 0; j < LA; ++j) a_off[j] = l_k + a_kc[j] < ke ? a_off[j] : kGemmOutside;
        }
        ars = gemm_descriptor(a_ptr, l_k < ke ? ((unsigned)a_rows * (unsigned)K - (unsigned)l_k) * 2u : 0u);
        const int64_t rem = w_rem < 0 ? 0 : w_rem;
        wrs = gemm_descriptor(w_ptr, (unsigned)(rem < kGemmMaxRecords ? rem : kGemmMaxRecords));
    };
    auto load_one = [&](int i) {  // load i of the stage
        if (i < LA)
            gemm_dma16<false>(ars, a_off[i < LA ? i : 0], l_dst + 1024u * (unsigned)(wave * LA + i));
        else
            gemm_dma16<NT>(wrs, w_off[i < LA ? 0 : i - LA], l_dst + 2u * AE + 1024u * (unsigned)(wave * LW + i - LA));
    };
    auto end_stage = [&]() {
        a_ptr += kGemmBK;
        w_ptr += (int64_t)kGemmBK * N;
        w_rem -= (int64_t)kGemmBK * N * 2;
        l_k += kGemmBK;
        l_dst += 2u * SE;
        if (l_dst == lds0 + S * 2u * SE) l_dst = lds0;
    };
    auto load_stage = [&]() {
        begin_stage();
#pragma unroll
        for (int i = 0; i < LS; ++i) load_one(i);
        end_stage();
    };

    const int wm = wave / WN, wn = wave % WN;
    const int r32 = lane & 31, h = lane >> 5, i16 = lane & 15, dsub = (lane >> 4) & 1;
    int a_at[4], b_at[NB];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a_at[kk] = gemm_a_slot(wm * (BM / WM) + r32, 2 * kk + h);
#pragma unroll
    for (int bn = 0; bn < NB; ++bn) {
        const int r = 8 * h + (i16 >> 2);  // +16 kk and +4 keep the row's permutation
        const int col = wn * (BN / WN) + bn * 32 + dsub * 16 + (i16 & 3) * 4;
        b_at[bn] = AE + r * BN + (((col >> 3) ^ wswz(r)) << 3) + (col & 7);
    }
    f32x16_t acc[MB][NB];
#pragma unroll
    for (int am = 0; am < MB; ++am)
#pragma unroll
        for (int bn = 0; bn < NB; ++bn) acc[am][bn] = f32x16_t{};
    bf16x8_t af[2][KC][MB], bf[2][KC][NB];

    constexpr int FR = KC * (MB + NB);  // fragments per cluster
    // fragment f of slices kk0 .. kk0 + KC - 1 of the stage at st, into set SET
    auto read_frag = [&](auto set_tag, const uint16_t* st, int kk0, int f) {
        constexpr int SET = decltype(set_tag)::value;
        const int k2 = f / (MB + NB), g = f - k2 * (MB + NB);
        // in the order of use: A block 0, the W blocks, the other A blocks
        if (g >= 1 && g <= NB) {
            const uint16_t* p = st + b_at[g >= 1 && g <= NB ? g - 1 : 0] + 16 * (kk0 + k2) * BN;
            const bf16x4_t b0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((gemm_lds_bf16x4_t*)(p));
            const bf16x4_t b1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((gemm_lds_bf16x4_t*)(p + 4 * BN));
            bf[SET][k2][g >= 1 && g <= NB ? g - 1 : 0] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
            const int am = g == 0 ? 0 : g - NB;
            af[SET][k2][am] = *reinterpret_cast<const bf16x8_t*>(st + a_at[kk0 + k2] + am * 32 * kGemmBK);
        }
    };
    // MFMAs of a cluster from set CUR; the next cluster's fragments and this cluster's share of the
    // loads ([L0, L1) of the stage being loaded) go between them
    auto cluster = [&](auto cur_tag, const uint16_t* st, int kk0, auto l0_tag, auto l1_tag) {
        constexpr int CUR = decltype(cur_tag)::value;
        constexpr int L0 = decltype(l0_tag)::value, L1 = decltype(l1_tag)::value;
        constexpr int NM = KC * MB * NB, NL = L1 - L0;
        // side work per MFMA: the loads at the last of each group of NM / NL gaps, the fragment
        // reads over the others
        constexpr int GAPS = NM > NL ? NM - NL : NM;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int k2 = i / (MB * NB), am = i / NB % MB, bn = i % NB;
            acc[am][bn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[CUR][k2][am], bf[CUR][k2][bn], acc[am][bn], 0, 0, 0);
            const int l0 = NL * i / NM, l1 = NL * (i + 1) / NM;  // loads of this gap
            const int g0 = NM > NL ? i - l0 : i, g1 = NM > NL ? i + 1 - l1 : i + 1;  // read gaps before and after it
#pragma unroll
            for (int f = FR * g0 / GAPS; f < FR * g1 / GAPS; ++f) read_frag(std::integral_constant<int, CUR ^ 1>{}, st, kk0, f);
#pragma unroll
            for (int l = l0; l < l1; ++l) load_one(L0 + l);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto meet = [&]() {  // the wave's fragment reads are done, its loads of the next stage have landed
        __builtin_amdgcn_s_waitcnt(wait_vmcnt_imm((S - 2) * LS) & ~0x0F00);
        ring_barrier();
    };
    using Z = std::integral_constant<int, 0>;
    using O = std::integral_constant<int, 1>;
    using LEnd = std::integral_constant<int, LS>;
    // Loads of a stage by cluster: the last cluster of a step starts a stage, the following ones
    // of the next step finish it.
    constexpr int Q = (LS + NC - 1) / NC;
    auto at = [](auto c_tag) { return std::integral_constant<int, (decltype(c_tag)::value * Q < LS ? decltype(c_tag)::value * Q : LS)>{}; };

#pragma unroll
    for (int i = 0; i < S - 1; ++i) load_stage();
    meet();
#pragma unroll
    for (int f = 0; f < FR; ++f) read_frag(Z{}, lds, 0, f);
    begin_stage();
    if (NC > 1) {
#pragma unroll
        for (int i = 0; i < (NC > 1 ? Q : 0); ++i) load_one(i);
    } else {
#pragma unroll
        for (int i = 0; i < LS; ++i) load_one(i);
        end_stage();
    }
    int slot = 0;  // of the ring, being read
    auto step = [&](auto par_tag) {
        constexpr int PAR = decltype(par_tag)::value;  // fragment set of the step's first cluster
        const uint16_t* cur = lds + slot * SE;
        slot = slot == S - 1 ? 0 : slot + 1;
        const uint16_t* nxt = lds + slot * SE;
        using P0 = std::integral_constant<int, PAR>;
        using P1 = std::integral_constant<int, PAR ^ 1>;
        using L2 = std::integral_constant<int, 2>;
        using L3 = std::integral_constant<int, 3>;
        if constexpr (NC == 1) {
            meet();
            begin_stage();
            cluster(P0{}, nxt, 0, Z{}, LEnd{});
            end_stage();
        } else if constexpr (NC == 2) {
            cluster(P0{}, cur, KC, at(O{}), LEnd{});
            end_stage();
            meet();
            begin_stage();
            cluster(P1{}, nxt, 0, Z{}, at(O{}));
        } else {
            cluster(P0{}, cur, 1, at(O{}), at(L2{}));
            cluster(P1{}, cur, 2, at(L2{}), at(L3{}));
            cluster(P0{}, cur, 3, at(L3{}), LEnd{});
            end_stage();
            meet();
            begin_stage();
            cluster(P1{}, nxt, 0, Z{}, at(O{}));
        }
    };
    if constexpr (NC == 1) {
        int t = 0;
        for (; t + 2 <= nk; t += 2) {
            step(Z{});
            step(O{});
        }
        if (t < nk) step(Z{});
    } else {
        for (int t = 0; t < nk; ++t) step(Z{});
    }

    if (EPI == kEpiPartial) {
        // fp32 products straight from the accumulators: for each e, 32 lanes store 128
        // contiguous bytes of one row
        float* out = P.partial + (int64_t)blockIdx.y * M * N;
#pragma unroll
        for (int am = 0; am < MB; ++am)
#pragma unroll
            for (int bn = 0; bn < NB; ++bn) {
                const int col = n0 + wn * (BN / WN) + bn * 32 + r32;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = m0 + wm * (BM / WM) + am * 32 + 8 * (e >> 2) + 4 * h + (e & 3);
                    if (row < M && col < N) out[(int64_t)row * N + col] = acc[am][bn][e];
                }
            }
        return;
    }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt_imm(0) & ~0x0F00);  // the loads past the k range have landed too
    ring_barrier();
    gemm_epilogue<BM, BN, WM, WN, EPI>(P, acc, lds, m0, n0);
}

constexpr int kGemmMaxSplits = 8;

// Sum over the splits of 8 partial products from element e0, in split order.  Every split's loads are
// requested before the first is added.
__device__ __forceinline__ void split_sum8(const float* __restrict__ partial, int splits, int64_t MN, int64_t e0, float (&v)[8]) {
    float4 lo[kGemmMaxSplits], hi[kGemmMaxSplits];
#pragma unroll
    for (int s = 0; s < kGemmMaxSplits; ++s) {
        if (s < splits) {  // uniform
            lo[s] = *reinterpret_cast<const float4*>(partial + s * MN + e0);
            hi[s] = *reinterpret_cast<const float4*>(partial + s * MN + e0 + 4);
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = 0.f;
#pragma unroll
    for (int s = 0; s < kGemmMaxSplits; ++s) {
        if (s < splits) {
            v[0] += lo[s].x; v[1] += lo[s].y; v[2] += lo[s].z; v[3] += lo[s].w;
            v[4] += hi[s].x; v[5] += hi[s].y; v[6] += hi[s].z; v[7] += hi[s].w;
        }
    }
}

__device__ __forceinline__ u32x4_t round8(const float (&v)[8]) {
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        o[i] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v[2 * i]) |
               ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)v[2 * i + 1]) << 16);
    return o;
}

// D = round(sum over splits of partial (+ D)), or silu(gate) * up of the rounded sums; 8 columns
// per thread (N % 8 == 0, N / 2 % 8 == 0 for SwiGLU, so a chunk stays in one row); grid-stride
// over the chunks of D.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(const float* __restrict__ partial, int splits,
                                                                uint16_t* __restrict__ D, int M, int N) {
    const int64_t MN = (int64_t)M * N;
    const int cpr = (EPI == kEpiSwiglu ? N / 2 : N) / 8;  // chunks per row of D
    const int64_t chunks = (int64_t)M * cpr;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < chunks; q += (int64_t)gridDim.x * 256) {
        const int64_t e0 = 8 * q;
        float v[8];
        if (EPI == kEpiSwiglu) {
            const int64_t row = q / cpr, at = row * N + 8 * (q - row * cpr);
            split_sum8(partial, splits, MN, at, v);
            const u32x4_t g = round8(v);
            split_sum8(partial, splits, MN, at + N / 2, v);
            *reinterpret_cast<u32x4_t*>(D + e0) = swiglu8(g, round8(v));
            continue;
        }
        split_sum8(partial, splits, MN, e0, v);
        if (EPI == kEpiAccumulate) {
            const u32x4_t d = *reinterpret_cast<const u32x4_t*>(D + e0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] += bf16_lo(d[i]);
                v[2 * i + 1] += bf16_hi(d[i]);
            }
        }
        *reinterpret_cast<u32x4_t*>(D + e0) = round8(v);
    }
}

// D[M, N / 2] = silu(gate) * up from the [gate | up] rows of gu[M, N]; grid-stride over chunks of 8.
__global__ __launch_bounds__(256) void swiglu_kernel(const uint16_t* __restrict__ gu, uint16_t* __restrict__ D, int M, int N) {
    const int cpr = N / 16;  // chunks per row of D
    const int64_t chunks = (int64_t)M * cpr;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < chunks; q += (int64_t)gridDim.x * 256) {
        const int64_t row = q / cpr;
        const uint16_t* g = gu + row * N + 8 * (q - row * cpr);
        *reinterpret_cast<u32x4_t*>(D + 8 * q) =
            swiglu8(*reinterpret_cast<const u32x4_t*>(g), *reinterpret_cast<const u32x4_t*>(g + N / 2));
    }
}

// ---------------------------------------------------------------- 256 x 256 tiles
// For grids that fill the chip: 8 waves (2 x 4) own a 256 x 256 tile, 128 x 64 each (4 x 2 MFMA
// blocks, 128 fp32 accumulators per lane), so the workgroup moves half the global bytes per flop of
// a 128 x 128 tile.  Bound: the matrix cores at the clock the part's power limit leaves them.
//   * K runs in half steps of 32.  A stages hold 64 k (whole 128-byte lines of A) in a ring of 3, W
//     stages 32 k in a ring of 4, together all 160 KB of LDS.
//   * The loads (64 of 1 KB per 64 k and workgroup, ~16 cycles each on the load path) go out between
//     the MFMAs, 4 per wave and half step; issued together at the start of a step they held up every
//     wave's first MFMA by ~1000 of its 2048 cycles.  A load has two half steps (2048 MFMA cycles of
//     a SIMD) to land.
//   * Fragments are read one 16-wide k slice ahead, one after each MFMA.  The workgroup meets between
//     the two slices of half step h: there every wave has read all of W half-stage h (and, for odd h,
//     of its A stage) and has waited for its loads of half-stage h + 1.
// Measured at 32768 x 4096 x 12288 (random bf16), against two 64 KB stages loaded at the start of a step:
// 2825 -> 2650 us (1.17 -> 1.24 PFLOP/s), timed in turn; cycles per launch 5.03 -> 4.26 million per XCD (MFMA busy
// 62.6 -> 73.8%), at a clock that falls from 1.81 to 1.60 GHz.
constexpr int kG2BM = 256;
constexpr int kG2BN = 256;
constexpr int kG2BK = 64;                              // k per A stage; a W half-stage holds 32
constexpr int kG2Waves = 8;
constexpr int kG2Threads = kG2Waves * 64;
constexpr int kG2AStages = 3;                          // A ring: 3 x 32 KB
constexpr int kG2WHalves = 4;                          // W ring: 4 x 16 KB
constexpr int kG2AElems = kG2BM * kG2BK;
constexpr int kG2WElems = 32 * kG2BN;
constexpr int kG2LdsElems = kG2AStages * kG2AElems + kG2WHalves * kG2WElems;  // 160 KB, all of it
static_assert(kG2LdsElems * 2 <= 160 * 1024, "LDS");

__device__ __forceinline__ int g2_w_slot(int r, int c) { return r * kG2BN + ((c ^ ((r & 3) << 2)) << 3); }

template <int EPI>
__global__ __launch_bounds__(kG2Threads, 1) void gemm_tile256_kernel(GemmParams P) {
    __shared__ __attribute__((aligned(1024))) uint16_t lds[kG2LdsElems];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int m0, n0;
    gemm_tile_origin(P, kG2BM, EPI == kEpiSwiglu ? kG2BN / 2 : kG2BN, m0, n0);
    const int M = P.M, N = P.N, K = P.K;
    const unsigned lds0 = (unsigned)(size_t)((gemm_lds_void_t*)lds);

    const int a_rows = min(M - m0, kG2BM);
    unsigned a_off[4], w_off[2];
    int a_kc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // A half-stage i of wave w: rows 128 i + 16 w .. + 16, two loads of 8 rows
        const int ar = 128 * (j >> 1) + 16 * wave + 8 * (j & 1) + (lane >> 3);
        const int ac = (lane & 7) ^ ((ar >> 1) & 7);
        a_kc[j] = 8 * ac;
        a_off[j] = (unsigned)ar * (unsigned)K * 2u + 16u * (unsigned)ac;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {  // W half-stage of wave w: rows 4 w .. + 4, two loads of 2 rows
        const int wr = 4 * wave + 2 * j + (lane >> 5);
        const int wc = (lane & 31) ^ ((wr & 3) << 2);
        // SwiGLU: the tile's columns are 128 gate columns, then the up columns beside them
        const bool up = EPI == kEpiSwiglu && wc >= 16;
        const int col = up ? 8 * wc - kG2BN / 2 : 8 * wc;
        const bool in = n0 + col < (EPI == kEpiSwiglu ? N / 2 : N);
        w_off[j] = in ? ((unsigned)wr * (unsigned)N + (unsigned)(up ? col + N / 2 : col)) * 2u : kGemmOutside;
    }
    const int nk = (K + kG2BK - 1) / kG2BK;
    // running load positions (uniform)
    const uint16_t* a_ptr = P.A + (int64_t)m0 * K;  // of the next A stage to load
    int a_k = 0, a_slot = 0;
    const uint16_t* w_ptr = P.W + n0;
    int64_t w_rem = ((int64_t)K * N - n0) * 2;
    int w_slot = 0;
    const int64_t w_stride = (int64_t)32 * N * 2;
    auto load_a_half = [&](int half) {
        if (half == 0 && K - a_k < kG2BK) {  // the last, ragged stage (once): chunks past K go outside
#pragma unroll
            for (int j = 0; j < 4; ++j) a_off[j] = a_k + a_kc[j] < K ? a_off[j] : kGemmOutside;
        }
        const unsigned rec = a_k < K ? ((unsigned)a_rows * (unsigned)K - (unsigned)a_k) * 2u : 0u;
        const gemm_i32x4_t rs = gemm_descriptor(a_ptr, rec);
        const unsigned dst = lds0 + 2u * (unsigned)(a_slot * kG2AElems + (128 * half + 16 * wave) * kG2BK);
        gemm_dma16<false>(rs, a_off[2 * half], dst);
        gemm_dma16<false>(rs, a_off[2 * half + 1], dst + 1024u);
        if (half == 1) {
            a_ptr += kG2BK;
            a_k += kG2BK;
            a_slot = a_slot == kG2AStages - 1 ? 0 : a_slot + 1;
        }
    };
    auto load_w_half = [&]() {
        const int64_t r0 = w_rem < 0 ? 0 : w_rem;
        const gemm_i32x4_t rs = gemm_descriptor(w_ptr, (unsigned)(r0 < kGemmMaxRecords ? r0 : kGemmMaxRecords));
        const unsigned dst = lds0 + 2u * (unsigned)(kG2AStages * kG2AElems + w_slot * kG2WElems + 4 * wave * kG2BN);
        gemm_dma16<false>(rs, w_off[0], dst);
        gemm_dma16<false>(rs, w_off[1], dst + 1024u);
        w_ptr += (int64_t)32 * N;
        w_rem -= w_stride;
        w_slot = (w_slot + 1) & (kG2WHalves - 1);
    };

    const int wm = wave >> 2, wn = wave & 3;
    const int r32 = lane & 31, h = lane >> 5, i16 = lane & 15, dsub = (lane >> 4) & 1;
    const int a_row0 = (wm * 128 + r32) * kG2BK;
    int a_chunk[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) a_chunk[kk] = a_row0 + (((2 * kk + h) ^ ((r32 >> 1) & 7)) << 3);
    int b_off[2];
#pragma unroll
    for (int bn = 0; bn < 2; ++bn) {
        const int r = 8 * h + (i16 >> 2);
        const int col = wn * 64 + bn * 32 + dsub * 16 + (i16 & 3) * 4;
        b_off[bn] = kG2AStages * kG2AElems + g2_w_slot(r, col >> 3) + (col & 7);
    }
    f32x16_t acc[4][2];
#pragma unroll
    for (int am = 0; am < 4; ++am)
#pragma unroll
        for (int bn = 0; bn < 2; ++bn) acc[am][bn] = f32x16_t{};
    bf16x8_t af[2][4], bf[2][2];

    auto read_a = [&](const uint16_t* st, int kk, int am) {
        return *reinterpret_cast<const bf16x8_t*>(st + a_chunk[kk] + am * 32 * kG2BK);
    };
    auto read_b = [&](const uint16_t* st, int k2, int bn) {
        const uint16_t* p = st + b_off[bn] + 16 * k2 * kG2BN;
        const bf16x4_t b0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((gemm_lds_bf16x4_t*)(p));
        const bf16x4_t b1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((gemm_lds_bf16x4_t*)(p + 4 * kG2BN));
        return __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // 8 MFMAs of one 16-wide k slice from fragment set CUR; after each goes one piece of the side work
    auto cluster = [&](auto cur_tag, const uint16_t* ast, const uint16_t* wst, int kk, int k2, auto&& dma) {
        constexpr int CUR = decltype(cur_tag)::value;
        constexpr int NXT = CUR ^ 1;
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int am = i >> 1, bn = i & 1;
            acc[am][bn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[CUR][am], bf[CUR][bn], acc[am][bn], 0, 0, 0);
            if (i == 0) bf[NXT][0] = read_b(wst, k2, 0);
            if (i == 1) bf[NXT][1] = read_b(wst, k2, 1);
            if (i >= 2 && i < 6) af[NXT][i - 2] = read_a(ast, kk, i - 2);
            if (i == 3) dma();
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_setprio(0);
    };
    auto meet = [&]() {  // this wave's fragment reads are done, its loads but the last 8 have landed
        __builtin_amdgcn_s_waitcnt(0x0078 | (0 << 14));  // vmcnt 8, expcnt 7, lgkmcnt 0
        ring_barrier();
    };
    using Z = std::integral_constant<int, 0>;
    using O = std::integral_constant<int, 1>;

    load_a_half(0);
    load_a_half(1);
    load_w_half();
    load_w_half();
    load_a_half(0);
    load_w_half();
    load_a_half(1);
    __builtin_amdgcn_s_waitcnt(0x0078);
    ring_barrier();
    {
#pragma unroll
        for (int am = 0; am < 4; ++am) af[0][am] = read_a(lds, 0, am);
#pragma unroll
        for (int bn = 0; bn < 2; ++bn) bf[0][bn] = read_b(lds, 0, bn);
    }
    load_w_half();
    int ra = 0, rw = 0;  // ring slots being read
    for (int t = 0; t < nk; ++t) {
        const uint16_t* ast = lds + ra * kG2AElems;
        const int ra1 = ra == kG2AStages - 1 ? 0 : ra + 1;
        const uint16_t* ast1 = lds + ra1 * kG2AElems;
        const uint16_t* w0 = lds + rw * kG2WElems;
        const uint16_t* w1 = lds + ((rw + 1) & 3) * kG2WElems;
        const uint16_t* w2 = lds + ((rw + 2) & 3) * kG2WElems;
        cluster(Z{}, ast, w0, 1, 1, [&] { load_a_half(0); });
        meet();
        cluster(O{}, ast, w1, 2, 0, [&] { load_w_half(); });
        cluster(Z{}, ast, w1, 3, 1, [&] { load_a_half(1); });
        meet();
        cluster(O{}, ast1, w2, 0, 0, [&] { load_w_half(); });
        ra = ra1;
        rw = (rw + 2) & 3;
    }
    __builtin_amdgcn_s_waitcnt(0x0070);  // the loads past K (zeros) have landed too
    ring_barrier();

    gemm_epilogue<kG2BM, kG2BN, 2, 4, EPI>(P, acc, lds, m0, n0);
}

}  // namespace trajspec
