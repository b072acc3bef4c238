// binary32 grouped product of the expert FFN on the matrix cores: up to 32 or 64 rows of one expert x 64 columns per workgroup.
//
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in binary32.  The four wavefronts split k, so the k loop has no
// barrier: every wavefront streams its quarter of the rows and of the weights into registers, 64 k ahead, and the four partial tiles
// meet in LDS once at the end.
//   tokens   lane (g, c) of 4 x 16 wants 4 consecutive k (4g .. 4g+3) of row c, one k per instruction: through LDS where k
//            allows (f32_tile_staged), else straight from memory
//   weights  row-major as the caller keeps them: the lane loads columns 4c .. 4c+3 of each of its 4 k; column 4c + s is
//            column c of instruction strip s, so the 64 columns of the tile are 4 strips and every load is a 256-byte run
// 16-row blocks keep the padding of short slots small; blocks a tile does not have are not compiled into its body.
//
// Bound: few rows per expert by the weight stream (32 experts x 32 rows, 512 x 2048: 4.4 TB/s, 4.9 with no matrix work), many by the
// matrix pipes (8 x 512 rows, 768 x 3072: 100 of 120 TFLOP/s that the loop reaches without loads); between them by what the tiles load
// twice.  Both products, tokens straight from memory and as now, us (of the gain 1 .. 1.5 us per product are the search of ffn_share.h):
//   512 x 2048: 32 experts x 32 rows 69, 61; 40 slots of 10 .. 59 rows 119, 101; 8 x 256 rows 107, 95; 16 x 94 rows 112, 91
//   768 x 3072, 8 x 512 rows: 493, 400       256 x 1024, 8 experts, 300 rows 22.3, 16.7       64 x 256, 8 x 64 rows 12.9, 10.1
#pragma once
#include "ffn_share.h"
#include <type_traits>

namespace moe {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int F32_THREADS = SHARE_THREADS;
constexpr int F32_BN = 64, F32_NARROW_BN = 32;
constexpr int F32_LD = F32_BN + 4;
constexpr int F32_STAGED = 2;          // D of the kernel that stages its tokens: two steps of 32 k

// First k of wavefront w's step of 16.  It hangs on k alone, so that every kernel here sums a row in the same order: both schedules
// and every batch size give the same bits.  Past 256 the steps are dealt in pairs, where that comes out even: the four wavefronts then
// read on in neighbouring lines.  Else, and where a wavefront has no more than two pairs, each has a quarter of k.
// QUARTERS: k is known to be one of those.
template <bool QUARTERS>
__device__ __forceinline__ int f32_k(int K, int w, int step)
{
    if (QUARTERS) return w * (K / 4) + step * 16;
    const bool dealt = K > 256 && K % 128 == 0;                  // uniform
    return w * (dealt ? 32 : K / 4) + (step >> 1) * (dealt ? 128 : 32) + (step & 1) * 16;
}

// part[w] <- this wavefront's share of k of (16 * MB rows) x 64 columns.  D: steps of 16 k in flight (f32_depth below)
template <int MB, bool STREAM, int D, bool QUARTERS, int BLOCKS>
__device__ __forceinline__ void f32_tile(const float *const (&a_row)[BLOCKS], const float *__restrict__ B, int K, int N,
                                         float (*__restrict__ part)[F32_LD])
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, g = lane >> 4;
    const int steps = K / 64;                                    // per wavefront
    const unsigned b_lane = (unsigned)(4 * g) * N + 4 * c;
    const float *a_src[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) a_src[m] = a_row[m] + 4 * g;
    f32x4_t a[D][MB], b[D][4], acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[m][s] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    // every load is unconditional (past the end: a harmless re-read), so that the waits can be counts
    auto load = [&](int step, int j) {
        const int k0 = f32_k<QUARTERS>(K, w, step < steps ? step : steps - 1);      // scalar, as are the weight rows' addresses
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4_t *p = reinterpret_cast<const f32x4_t *>(B + (size_t)(k0 + i) * N + b_lane);
            b[j][i] = STREAM ? __builtin_nontemporal_load(p) : *p;
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) a[j][m] = *reinterpret_cast<const f32x4_t *>(a_src[m] + k0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int j) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j][m][i], b[j][i][s], acc[m][s], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int j = 0; j < D; ++j) load(j, j);
    int s = 0;
    for (; s + D < steps; s += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            multiply(j);
            load(s + D + j, j);
        }
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (s + j < steps) multiply(j);                          // uniform
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)                              // accumulator register i: row 4g + i, column c of strip s
            *reinterpret_cast<f32x4_t *>(&part[m * 16 + 4 * g + i][4 * c]) =
                (f32x4_t){acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]};
}

// The same share of k with the tokens staged through the wavefront's own piece of LDS (its part of `part`, which is written after the
// last step): a step is 32 k, a token load takes eight rows' 128 consecutive bytes, and the fragments (lane (g, c): row c, 4 k) are
// read back from there.  Loaded straight from memory a fragment touches 16 lines per 16 lanes and holds the load path four times as
// long as its bytes need.
constexpr int F32_LDA = 32 + 4;

// src: the rows this lane loads (tile rows lane / 8 + 8 i).
// gathered: they come from an index, a bad one reads row 0.
template <int MB, int NS, bool STREAM, int D, int ROWS>
__device__ __forceinline__ void f32_tile_staged(const float *__restrict__ A, const int (&src)[ROWS], bool gathered, int n_src_rows,
                                                const float *__restrict__ B, int K, int N, float (*__restrict__ part)[16 * NS + 4])
{
    typedef float strips_t __attribute__((ext_vector_type(NS)));    // neighbouring columns of a lane, one per strip
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, g = lane >> 4;
    const int steps = K / 128;                                   // per wavefront
    const unsigned b_lane = (unsigned)(4 * g) * N + NS * c;
    float *stage = &part[0][0];
    float *put = stage + (lane >> 3) * F32_LDA + (lane & 7) * 4;
    const float *get = stage + c * F32_LDA + 4 * g;
    f32x4_t a[D][2 * MB], acc[MB][NS];
    strips_t b[D][2][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int s = 0; s < NS; ++s) acc[m][s] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    auto k_of = [&](int step) { return f32_k<false>(K, w, 2 * (step < steps ? step : steps - 1)); };     // past the end: a harmless re-read
    auto load_b = [&](int step, int j) {
        const int k0 = k_of(step);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const strips_t *p = reinterpret_cast<const strips_t *>(B + (size_t)(k0 + 16 * h + i) * N + b_lane);
                b[j][h][i] = STREAM ? __builtin_nontemporal_load(p) : *p;
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    const float *a_row[2 * MB];
    auto load_a = [&](int step, int j) {
        const int k0 = k_of(step);
#pragma unroll
        for (int i = 0; i < 2 * MB; ++i) a[j][i] = *reinterpret_cast<const f32x4_t *>(a_row[i] + k0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto load = [&](int step, int j) {
        load_a(step, j);
        load_b(step, j);
    };
    auto multiply = [&](int j) {
        f32x4_t f[2][MB];
#pragma unroll
        for (int i = 0; i < 2 * MB; ++i) *reinterpret_cast<f32x4_t *>(put + i * 8 * F32_LDA) = a[j][i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS operations of one wavefront execute in order
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int m = 0; m < MB; ++m) f[h][m] = *reinterpret_cast<const f32x4_t *>(get + m * 16 * F32_LDA + 16 * h);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[h][m][i], b[j][h][i][s], acc[m][s], 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_sched_barrier(0);
    };

    const unsigned limit = gathered ? (unsigned)n_src_rows : 0x80000000u;       // a select per row, not a branch
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
        const int r = (unsigned)src[i] < limit ? src[i] : 0;
        a_row[i] = A + (size_t)r * K + (lane & 7) * 4;
    }
#pragma unroll
    for (int j = 0; j < D; ++j) load(j, j);
    int s = 0;
    for (; s + D < steps; s += D) {
#pragma unroll
        for (int j = 0; j < D; ++j) {
            multiply(j);
            load(s + D + j, j);
        }
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (s + j < steps) multiply(j);                          // uniform
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            strips_t v;
#pragma unroll
            for (int s = 0; s < NS; ++s) v[s] = acc[m][s][i];
            *reinterpret_cast<strips_t *>(&part[m * 16 + 4 * g + i][NS * c]) = v;
        }
}

// SEVERAL: units per workgroup (f32_grid); else one, which is up to 5 % faster with nothing kept for the next
// OUT: the layer's output too (LayerOut); the token of a row is asked for before the product, its probability and x after it
template <bool RELU, int BM, int BN, int D, bool SEVERAL, bool OUT = false>
__global__ __launch_bounds__(F32_THREADS, BM == 32 ? 3 : 2) void ffn_gemm_f32_kernel(
    const float *__restrict__ A, const float *__restrict__ W, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int max_rows, float *__restrict__ C, LayerOut layer)
{
    __shared__ __attribute__((aligned(16))) float part[4][BM][BN + 4];
    __shared__ TileItem found;
    TileShare<BM> share;
    share.E = E;
    share.schedule = schedule;
    share.n_nt = N / BN;
    share.max_rows = max_rows;
    const int tid = threadIdx.x, w = tid >> 6, c = tid & 15;
    LayerOut::Deal dropped;
    if constexpr (OUT) dropped = layer.deal_dropped(N / 4);
    share.find(slot_offset, slot_expert, n_slots_p, max_slots, &found);
    if constexpr (OUT) layer.copy_dropped(dropped, N / 4);
    for (int unit = share.first + (int)(blockIdx.x >> 3); unit < share.end; unit += (int)(gridDim.x >> 3)) {      // uniform
        share.write_item(slot_offset, slot_expert, unit, &found);
        __syncthreads();
        const TileItem it = found;
        const bool good = it.expert >= 0 && it.expert < E && it.row_begin >= 0;       // uniform; never index with a bad table
        const int nt = it.column;
        const float *B = W + (size_t)it.expert * K * N + nt * BN;
        const int row_end = !good ? it.row_begin : it.row_end < max_rows ? it.row_end : max_rows;
        for (int r0 = it.row_begin; r0 < row_end; r0 += BM) {
            const int nrows = row_end - r0 < BM ? row_end - r0 : BM;
            // the rows this lane loads: row c of every block, or (staged) every eighth row of the tile
            constexpr int LOADS = D == F32_STAGED ? BM / 8 : BM / 16;
            const int l_row = D == F32_STAGED ? (tid & 63) >> 3 : c;
            int src[LOADS];
#pragma unroll
            for (int m = 0; m < LOADS; ++m) {                    // rows past the tile repeat its last row
                const int r = m * (BM / LOADS) + l_row;
                src[m] = r0 + (r < nrows ? r : nrows - 1);
            }
            if (row_index) {
#pragma unroll
                for (int m = 0; m < LOADS; ++m) src[m] = row_index[src[m]];
                if constexpr (D != F32_STAGED) {                 // a bad index reads row 0 (the staged tile sees to it itself)
#pragma unroll
                    for (int m = 0; m < LOADS; ++m) src[m] = src[m] >= 0 && src[m] < n_src_rows ? src[m] : 0;
                }
            }
            constexpr int ROWS_AT_ONCE = F32_THREADS / (BN / 4), ROWS = BM / ROWS_AT_ONCE;      // of the tile's epilogue
            const int r_first = tid / (BN / 4);
            int token[ROWS];
            if constexpr (OUT) {
#pragma unroll
                for (int i = 0; i < ROWS; ++i) {
                    const int r = r_first + i * ROWS_AT_ONCE;
                    token[i] = layer.perm[r0 + (r < nrows ? r : nrows - 1)];
                }
            }
            const int blocks = (nrows + 15) >> 4;
            auto tile = [&](auto BLOCKS, auto STREAM) {
                constexpr int M = decltype(BLOCKS)::value;
                constexpr bool S = decltype(STREAM)::value;
                if constexpr (D == F32_STAGED) {
                    f32_tile_staged<M, BN / 16, S, D>(A, src, row_index != nullptr, n_src_rows, B, K, N, part[w]);
                } else {
                    const float *a_row[LOADS];
#pragma unroll
                    for (int m = 0; m < LOADS; ++m) a_row[m] = A + (size_t)src[m] * K;
                    f32_tile<M, S, D, SEVERAL>(a_row, B, K, N, part[w]);
                }
            };
            using std::integral_constant;
#define MOE_F32_TILE(M)                                                        \
    do {                                                                       \
        if (it.reuse) tile(integral_constant<int, M>{}, std::false_type{});    \
        else tile(integral_constant<int, M>{}, std::true_type{});              \
    } while (0)
            if (blocks == 1) MOE_F32_TILE(1);
            else if (BM == 32 || blocks == 2) MOE_F32_TILE(2);
            else if constexpr (BM > 32) {
                if (blocks == 3) MOE_F32_TILE(3);
                else MOE_F32_TILE(4);
            }
#undef MOE_F32_TILE
            __syncthreads();
            const int col = tid % (BN / 4) * 4;
            float prob[ROWS];
            f32x4_t base[ROWS];
            if constexpr (OUT) {
#pragma unroll
                for (int i = 0; i < ROWS; ++i) {
                    token[i] = (unsigned)token[i] < (unsigned)layer.T ? token[i] : 0;
                    prob[i] = layer.prob[token[i]];
                    base[i] = layer.residual ? *reinterpret_cast<const f32x4_t *>(static_cast<const float *>(layer.x) + (size_t)token[i] * N + nt * BN + col)
                                             : (f32x4_t){0.f, 0.f, 0.f, 0.f};
                }
            }
            auto finish = [&](int r, int n) {                        // n: of this thread's rows
                f32x4_t p[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[q] = *reinterpret_cast<const f32x4_t *>(&part[q][r][col]);
                f32x4_t o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = (p[0][i] + p[1][i]) + (p[2][i] + p[3][i]);
                    o[i] = RELU ? fmaxf(v, 0.f) : v;
                }
                *reinterpret_cast<f32x4_t *>(C + (size_t)(r0 + r) * N + nt * BN + col) = o;
                if constexpr (OUT) {
                    f32x4_t v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = fmaf(prob[n], o[i], base[n][i]);
                    *reinterpret_cast<f32x4_t *>(static_cast<float *>(layer.out) + (size_t)token[n] * N + nt * BN + col) = v;
                }
            };
            if constexpr (OUT) {
#pragma unroll
                for (int n = 0; n < ROWS; ++n) {
                    const int r = r_first + n * ROWS_AT_ONCE;
                    if (r >= nrows) break;
                    finish(r, n);
                }
            } else {                                                 // rolled up: unrolled, these builds took up to 4 registers more or spilled 2
                for (int r = r_first; r < nrows; r += ROWS_AT_ONCE) finish(r, 0);
            }
            __syncthreads();
        }
        if (!SEVERAL) break;
        __syncthreads();                                             // found has been read by all
        if (tid == 0) found.expert = -1;
        __syncthreads();
    }
}

// Steps of 16 k per wavefront in flight: four, which a k of under 256 does not have (they would be asked for past its end all the same).
// There a unit is so short that finding it takes as long: tiles of 32 rows, several units per workgroup (f32_grid).  16384 rows over
// 128 experts, 64 -> 1024 -> 64, both products: 181 us with four steps and 64 rows, 165 with one, 118 with several units, 98 with 32 rows
// (111 with the kernel before).
static inline int f32_depth(int K) { return K < 256 ? 1 : 4; }

// Tile height of the others.  64 rows load a third less per multiply-add, 32 rows leave no CU with twice the tiles of another: few
// rows per expert make few tiles, and from 128 on average on there are enough of them (both products, us, with 64 and 32 rows:
// 768 x 3072, 8 experts x 512 rows 399, 428; 512 x 2048, 8 x 256 95, 102; 40 slots of 10 .. 59 rows 94, 91; 1300 rows by Zipf's law over
// 32 experts 136, 116).
static inline int f32_rows(int max_rows, int E) { return (long long)max_rows >= 128LL * E ? 64 : 32; }

// A workgroup per unit, except up to k = 256, where a unit is short beside its search: there twice as many as are resident (two with 64
// rows, three with 32) at most, and four per CU with the shortest k.  16384 rows over 128 experts, 256 -> 1024 -> 256: 308 -> 271 us;
// with longer k that deal leaves CUs idle at the end (8 experts, 512 -> 2048 -> 512: 743 -> 896 us).
static inline bool f32_several(int K) { return K <= 256; }
static inline int f32_grid(int bm, int max_rows, int max_slots, int schedule, int K, int N)
{
    const int all = share_grid(bm ? bm : 32, F32_BN, max_rows, max_slots, schedule, N);
    const int most = 256 * (bm == 0 ? 4 : bm == 64 ? 2 * 2 : 2 * 3);
    return !f32_several(K) || all < most ? all : most;
}

// Tokens through LDS wherever a wavefront's share of k is whole steps of 32.  At k = 256 there are two of them, and the loads they save
// are no longer than what the second unit of a workgroup needs (256 -> 1024 -> 256, 32 x 64 rows: 37.2 us without, 39.1 with).
// Nor where units of 64 rows, or (experts schedule) of several tiles, are so few that each has a CU for itself: then the load path is
// not what binds, and loads straight to registers come back sooner.  Both products, us, with LDS and without: 512 -> 2048 -> 512,
// 1 expert, 256 rows 55.4, 52.1, 512 rows 56.7, 52.6; 1024 -> 1024 -> 1024, 512 rows over 2 46.8, 43.8; experts schedule, 512 -> 2048 -> 512,
// 1024 rows over 8 302, 283.  The line of the slot schedule is low because the last tiles of the experts are cheap and crowd an XCD: 768 ->
// 3072 -> 768, 300 rows of 1 expert (240 units) 85, 89; 384 -> 1536 -> 384, 400 rows over 2 (192) 46.7, 52.4; 1024 -> 1024 -> 1024, 800 over 4 (256)
// 67, 98.
static inline bool f32_staged(int bm, int max_rows, int max_slots, int E, int schedule, int K, int N)
{
    if (f32_several(K) || K % 128 != 0) return false;
    const long long experts = max_slots < E ? max_slots : E;
    if (schedule == MOE_SCHEDULE_SLOTS) return bm == 32 || (max_rows / bm + experts) * (N / F32_BN) > 160;
    return max_rows <= 32 || experts * (N / F32_BN) > 256;
}

// 32 columns where 64 would leave at least half of the CUs without a unit: half the work per unit, but every token row is loaded twice as often.
// Both products, 64 and 32 columns, us: 256 -> 1024 -> 256, 300 rows over 8 experts 21.4 and 17.0; 512 -> 2048 -> 512, 200 over 16
// 42.6 and 43.8; 512 over 8 48.4 and 56.8.
static inline bool f32_narrow(int max_rows, int max_slots, int E, int schedule, int K, int N)
{
    const long long tiles = max_rows / 32 + (max_slots < E ? max_slots : E);
    return schedule == MOE_SCHEDULE_SLOTS && K >= 256 && K % 128 == 0 && f32_rows(max_rows, E) == 32 && tiles * (N / F32_BN) <= 128;
}
static inline int f32_narrow_grid(int max_rows, int max_slots, int schedule, int N)
{
    return share_grid(32, F32_NARROW_BN, max_rows, max_slots, schedule, N);
}

}  // namespace moe
