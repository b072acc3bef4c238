// bf16 matrix-core tile product for gfx950, shared by the expert FFN, the router and the SRU
// projections.
//
//   C[BM x BN] (fp32 accumulators) += A[rows, K] (row-major bf16, k contiguous) * B[K, N]
//
// B is read from the packed image (see moe_pack_weights): columns are grouped in strips of
// 32; inside a strip, for every group of 8 consecutive k, the 32 columns follow each other
// with their 8 k-values contiguous (16 bytes).  uint4 index of (k/8 = g, column n):
//     ((n/32) * (K/8) + g) * 32 + n%32
// The B operand of v_mfma_f32_32x32x16_bf16 wants, per lane, 8 consecutive k of one column
// (lanes 0-31: k 0-7, lanes 32-63: k 8-15 of the 16-deep step): in this image that is ONE
// 16-byte load per lane, the 64 lanes of a wavefront reading 1 KB of consecutive memory, and
// a wavefront walking down K reads one strip front to back.  Weights therefore stream from
// HBM straight into registers exactly once per workgroup, in DRAM-page order, and never
// pass through LDS.
//
// One workgroup = 4 wavefronts side by side along the columns.  Wavefront w owns MB row blocks of 32 rows and NB
// column strips (columns n0 + (w*NB + nb)*32 ..): MB*NB accumulators of 16 VGPRs, so every weight byte is loaded by
// exactly one wavefront.
// The A rows (tokens) are shared by the four wavefronts and staged through two LDS buffers in BK-wide k
// chunks.  Both operands are requested two chunks ahead: the registers of chunk i are refilled with chunk i+2 right after
// its matrix instructions, so two register sets hold two chunks in flight.
// Every load of the k loop is unconditional and the last chunks are peeled: where a load may or may not have been issued
// (a lane-masked row, an "if there is another chunk"), the compiler cannot count what is outstanding and waits for the
// youngest loads with the oldest -- each chunk then stalls for the prefetch it has just issued.  The requests of a chunk go
// out in one burst: spread between the matrix instructions, the same loads streamed at 5.3 instead of 6.4 TB/s.
// Measured against that (first, second product, us): 24 experts of 2 rows, 768 x 3072: 25.9, 29.4 -> 24.4, 23.2; 32 x 20 rows,
// 512 x 2048: 17.9, 21.4 -> 16.2, 17.4; 36 x 100 rows: 47.6, 50.6 -> 44.8, 41.6; 144 x 17 rows: 105, 113 -> 103, 108.
#pragma once
#include "common.h"
#include <type_traits>

namespace moe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int GEMM_THREADS = 256;

template <int MB, int BK>
constexpr int gemm_lds_elems()
{
    return 2 * MB * 32 * (BK + 8);   // row stride BK+8 elements keeps the b128 reads conflict free
}

// Row of accumulator register v (0..15) of a 32x32 block for this lane; its column is lane & 31.
__device__ __forceinline__ int acc_row(int v, int lane) { return 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }

// A: pointer to row 0 of the tile (already offset by the tile's first row); rows >= nrows repeat row nrows - 1 (the
// caller does not use what they give).
// row_idx (optional, already offset to the tile's first row): tile row r is read from
//   A + row_idx[r]*lda instead of A + r*lda (fused gather of token rows); an index outside [0, n_src_rows) reads row 0.
// Bp: packed matrix (K x N) of this tile's expert; n0 = first column of the tile (multiple of 32).
// K must be a multiple of BK.
// STREAM_B: the B operand is read exactly once in the whole launch (expert weights): load it
// with the non-temporal hint so the stream does not evict the activations the other operand
// and the epilogue keep in cache.  (Measured on the 604 MB weight stream of a 128-expert
// layer: 120 -> 110 us for the first FFN product, 111 -> 101 us for the second.)
template <int MB, int NB, int BK, bool STREAM_B = false>
__device__ __forceinline__ void gemm_tile_bf16(const bf16_t *__restrict__ A, int lda, int nrows,
                                               const bf16_t *__restrict__ Bp, int n0, int K,
                                               bf16_t *__restrict__ lds, f32x16_t (&acc)[MB][NB],
                                               const int32_t *__restrict__ row_idx = nullptr, int n_src_rows = 0)
{
    constexpr int LDA = BK + 8;
    constexpr int KS = BK / 16;                       // 16-deep MFMA steps per chunk
    constexpr int BM = MB * 32;                       // rows of the workgroup tile
    constexpr int PIECES = BM * (BK / 8);             // 16-byte pieces of one A chunk
    constexpr int A_PER_THREAD = PIECES / GEMM_THREADS;
    constexpr int ROW_STEP = GEMM_THREADS / (BK / 8);
    static_assert(PIECES % GEMM_THREADS == 0, "A chunk must split evenly over the workgroup");
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = K / BK;
    const int KG = K >> 3;
    typedef unsigned u32x4v_t __attribute__((ext_vector_type(4)));
    u32x4v_t a_reg[2][A_PER_THREAD];
    u32x4v_t b[2][KS][NB];
    const int a_col = tid % (BK / 8);
    const int a_row = tid / (BK / 8);
    // scalar address, the lane's own piece as the offset: one register instead of a pair per load
    const u32x4v_t *b_base = reinterpret_cast<const u32x4v_t *>(Bp) + (size_t)((n0 >> 5) + w * NB) * KG * 32;

    const bf16_t *a_src[A_PER_THREAD];   // this thread's rows stay the same for every k chunk
    auto load_a = [&](int kc, int set) {
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i) a_reg[set][i] = *reinterpret_cast<const u32x4v_t *>(a_src[i] + kc * BK);
    };
    auto load_b = [&](int kc, int set, int ks) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const u32x4v_t *p = b_base + ((size_t)nb * KG + kc * (BK / 8) + ks * 2) * 32 + lane;
            b[set][ks][nb] = STREAM_B ? __builtin_nontemporal_load(p) : *p;
        }
    };
    auto store_a = [&](int buf, int set) {
        bf16_t *dst = lds + buf * (BM * LDA);
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i)
            *reinterpret_cast<u32x4v_t *>(dst + (a_row + i * ROW_STEP) * LDA + a_col * 8) = a_reg[set][i];
    };
    // requests of a chunk, always in this order: the waits are counts, and one count has to fit the way into the loop
    // and the way round it
    auto request = [&](int kc, int set) {
        load_a(kc, set);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            load_b(kc, set, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // one pipeline stage: multiply chunk kc (register set and LDS buffer SET = kc & 1), request chunk kc + 2 into the
    // registers as they fall free, put chunk kc + 1 of the tokens into LDS
    auto stage = [&](int kc, auto SET, auto ISSUE, auto LAST) {
        constexpr int set = decltype(SET)::value;
        constexpr bool issue = decltype(ISSUE)::value;
        const bf16_t *src = lds + set * (BM * LDA) + (lane & 31) * LDA + (lane >> 5) * 8;
        u32x4v_t af[2][MB];              // fragments of this 16-deep step and the next
        auto read_a = [&](int ks) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) af[ks & 1][mb] = *reinterpret_cast<const u32x4v_t *>(src + mb * 32 * LDA + ks * 16);
        };
        read_a(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) read_a(ks + 1);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[ks & 1][mb]),
                                                                          __builtin_bit_cast(bf16x8_t, b[set][ks][nb]),
                                                                          acc[mb][nb], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (issue) request(kc + 2, set);
        if constexpr (!decltype(LAST)::value) store_a(set ^ 1, set ^ 1);
        __syncthreads();
    };
    using yes = std::true_type;
    using no = std::false_type;
    using even = std::integral_constant<int, 0>;
    using odd = std::integral_constant<int, 1>;

    // The first chunk's weights are on their way before the row numbers they do not depend on have arrived.  From the first
    // chunk's tokens on the order is the loop's.
    int rows[A_PER_THREAD];
#pragma unroll
    for (int i = 0; i < A_PER_THREAD; ++i) {
        const int r = a_row + i * ROW_STEP;
        rows[i] = r < nrows ? r : nrows - 1;
    }
    if (row_idx) {
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i) rows[i] = row_idx[rows[i]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) load_b(0, 0, ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < A_PER_THREAD; ++i) rows[i] = (rows[i] >= 0 && rows[i] < n_src_rows) ? rows[i] : 0;
    } else {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) load_b(0, 0, ks);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < A_PER_THREAD; ++i) a_src[i] = A + (size_t)rows[i] * lda + a_col * 8;
    load_a(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    request(nk > 1 ? 1 : 0, 1);
    store_a(0, 0);
    __syncthreads();
    int kc = 0;
    for (; kc + 3 < nk; kc += 2) {
        stage(kc, even{}, yes{}, no{});
        stage(kc + 1, odd{}, yes{}, no{});
    }
    // 1 .. 3 chunks are left.  The marks keep the three ways apart: their common first LDS reads would be moved in front
    // of the branch, into 64 registers that nothing else can spare
    if (nk - kc == 3) {
        asm volatile("; three chunks left" ::: "memory");
        stage(kc, even{}, yes{}, no{});
        stage(kc + 1, odd{}, no{}, no{});
        stage(kc + 2, even{}, no{}, yes{});
    } else if (nk - kc == 2) {
        asm volatile("; two chunks left" ::: "memory");
        stage(kc, even{}, no{}, no{});
        stage(kc + 1, odd{}, no{}, yes{});
    } else {
        asm volatile("; one chunk left" ::: "memory");
        stage(kc, even{}, no{}, yes{});
    }
}

template <int MB, int NB>
__device__ __forceinline__ void zero_acc(f32x16_t (&acc)[MB][NB])
{
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.f;
}

}  // namespace moe
