// binary32 grouped product of the expert FFN on the matrix cores: up to 32 or 64 rows of one expert x 64 columns per workgroup.
//
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in binary32.  The four wavefronts split k, so the k loop has no LDS and
// no barrier: every wavefront streams its quarter of the rows and of the weights straight into registers, D steps of 16 k
// ahead, and the four partial tiles meet in LDS once at the end.
//   tokens   lane (g, c) of 4 x 16 loads 4 consecutive k (4g .. 4g+3) of row c: one k per instruction
//   weights  row-major as the caller keeps them: the lane loads columns 4c .. 4c+3 of each of its 4 k; column 4c + s is
//            column c of instruction strip s, so the 64 columns of the tile are 4 strips and every load is a 256-byte run
// 16-row blocks keep the padding of short slots small; blocks a tile does not have are not compiled into its body.
//
// Bound: load time and matrix time add up.  A 32 x 64 tile loads 24 KB per 16 k, where its matrix instructions take 1024 clocks; with
// either left out 8 experts x 512 rows, 768 x 3072, take 128 and 161 us, with both 305.  Together the loads come in at about 55 GB/s per CU (a
// CU takes 135 GB/s of plain loads from its L2).  Measured (first, second product; the vector-unit tile before, 64 x 64 with
// both operands in LDS and one workgroup's whole k in one chain, in brackets): 32 experts x 32 rows, 512 x 2048: 43, 32 us (62, 102);
// 40 slots of 10 .. 59 rows: 66, 75 us (83, 140); 8 experts x 512 rows, 768 x 3072: 215, 279 us (249, 287).
#pragma once
#include "ffn_share.h"

namespace moe {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int F32_THREADS = SHARE_THREADS;
constexpr int F32_BN = 64;
constexpr int F32_LD = F32_BN + 4;

// part[w] <- this wavefront's share of k of (16 * MB rows) x 64 columns.  D: steps of 16 k in flight (f32_depth below)
template <int MB, bool STREAM, int D, int BLOCKS>
__device__ __forceinline__ void f32_tile(const float *const (&a_row)[BLOCKS], const float *__restrict__ B, int K, int N,
                                         float (*__restrict__ part)[F32_LD])
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, g = lane >> 4;
    const int steps = K / 64;                                    // per wavefront
    const int k_wave = w * (K / 4);                              // scalar, as are the weight rows' addresses
    const unsigned b_lane = (unsigned)(4 * g) * N + 4 * c;
    const float *a_src[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) a_src[m] = a_row[m] + k_wave + 4 * g;
    f32x4_t a[D][MB], b[D][4], acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[m][s] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    // every load is unconditional (past the end: a harmless re-read), so that the waits can be counts
    auto load = [&](int step, int j) {
        const int s = step < steps ? step : steps - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const f32x4_t *p = reinterpret_cast<const f32x4_t *>(B + (size_t)(k_wave + s * 16 + i) * N + b_lane);
            b[j][i] = STREAM ? __builtin_nontemporal_load(p) : *p;
        }
#pragma unroll
        for (int m = 0; m < MB; ++m) a[j][m] = *reinterpret_cast<const f32x4_t *>(a_src[m] + s * 16);
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

// SEVERAL: units per workgroup (f32_grid); else one, which is up to 5 % faster with nothing kept for the next
template <bool RELU, int BM, int D, bool SEVERAL>
__global__ __launch_bounds__(F32_THREADS, BM == 32 ? 3 : 2) void ffn_gemm_f32_kernel(
    const float *__restrict__ A, const float *__restrict__ W, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int max_rows, float *__restrict__ C)
{
    __shared__ __attribute__((aligned(16))) float part[4][BM][F32_LD];
    __shared__ TileItem found;
    TileShare<BM> share;
    share.E = E;
    share.schedule = schedule;
    share.n_nt = N / F32_BN;
    share.max_rows = max_rows;
    share.find(slot_offset, slot_expert, n_slots_p, max_slots);
    const int tid = threadIdx.x, w = tid >> 6, c = tid & 15;
    for (int unit = share.first + (int)(blockIdx.x >> 3); unit < share.end; unit += (int)(gridDim.x >> 3)) {      // uniform
        if (tid == 0) found.expert = -1;                             // stays so if the slot tables contradict themselves
        __syncthreads();
        share.write_item(slot_offset, slot_expert, unit, &found);
        __syncthreads();
        const TileItem it = found;
        if (it.expert < 0 || it.expert >= E || it.row_begin < 0) {               // uniform; never index with a bad table
            if (!SEVERAL) break;
            __syncthreads();                                         // found is read before the next unit's
            continue;
        }
        const int nt = it.column;
        const float *B = W + (size_t)it.expert * K * N + nt * F32_BN;
        const int row_end = it.row_end < max_rows ? it.row_end : max_rows;
        for (int r0 = it.row_begin; r0 < row_end; r0 += BM) {
            const int nrows = row_end - r0 < BM ? row_end - r0 : BM;
            int src[BM / 16];
#pragma unroll
            for (int m = 0; m < BM / 16; ++m)                    // rows past the tile repeat its last row
                src[m] = r0 + (m * 16 + c < nrows ? m * 16 + c : nrows - 1);
            if (row_index) {
#pragma unroll
                for (int m = 0; m < BM / 16; ++m) src[m] = row_index[src[m]];
#pragma unroll
                for (int m = 0; m < BM / 16; ++m)                // a bad index reads row 0
                    src[m] = src[m] >= 0 && src[m] < n_src_rows ? src[m] : 0;
            }
            const float *a_row[BM / 16];
#pragma unroll
            for (int m = 0; m < BM / 16; ++m) a_row[m] = A + (size_t)src[m] * K;
            const int blocks = (nrows + 15) >> 4;
#define MOE_F32_TILE(M)                                               \
    do {                                                              \
        if (it.reuse) f32_tile<M, false, D>(a_row, B, K, N, part[w]); \
        else f32_tile<M, true, D>(a_row, B, K, N, part[w]);           \
    } while (0)
            if (blocks == 1) MOE_F32_TILE(1);
            else if (BM == 32 || blocks == 2) MOE_F32_TILE(2);
            else if constexpr (BM > 32) {
                if (blocks == 3) MOE_F32_TILE(3);
                else MOE_F32_TILE(4);
            }
#undef MOE_F32_TILE
            __syncthreads();
            for (int r = tid >> 4; r < nrows; r += 16) {
                f32x4_t p[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) p[q] = *reinterpret_cast<const f32x4_t *>(&part[q][r][4 * c]);
                f32x4_t o;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v = (p[0][i] + p[1][i]) + (p[2][i] + p[3][i]);
                    o[i] = RELU ? fmaxf(v, 0.f) : v;
                }
                *reinterpret_cast<f32x4_t *>(C + (size_t)(r0 + r) * N + nt * F32_BN + 4 * c) = o;
            }
            __syncthreads();
        }
        if (!SEVERAL) break;
    }
}

// Steps of 16 k per wavefront in flight: four, which a k of under 256 does not have (they would be asked for past its end all the same).
// There a unit is so short that finding it takes as long: tiles of 32 rows, several units per workgroup (f32_grid).  16384 rows over
// 128 experts, 64 -> 1024 -> 64, both products: 181 us with four steps and 64 rows, 165 with one, 118 with several units, 98 with 32 rows
// (111 with the kernel before).
static inline int f32_depth(int K) { return K < 256 ? 1 : 4; }

// Tile height of the others.  64 rows load a third less per multiply-add, 32 rows leave no CU with twice the tiles of another: few
// rows per expert make few tiles, and from 128 on average on there are enough of them (8 experts x 512 rows, 768 x 3072:
// 215, 279 us against 248, 318 with 32 rows; 40 slots of 10 .. 59 rows, 512 x 2048: 80, 114 against 66, 75).
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

}  // namespace moe
