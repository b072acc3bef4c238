// bf16 grouped product for batches that leave most of the chip idle in the 128-column kernel: a decode step has rows for a
// few experts only, and 22 experts x 6 column tiles are 132 workgroups that each pull 786 KB, where a CU pulls about 55 GB/s.
//
// Up to 32 rows of one expert x 32 columns per workgroup, the four wavefronts split k: four times as many workgroups, and
// no LDS and no barrier in the k loop.  Each wavefront streams its quarter of one 32-column strip of the packed image (1 KB of
// consecutive memory per load, already the matrix-core operand) and the token rows next to it straight into registers, 12
// steps of 16 k ahead, refilled in bursts of 4; the partial tiles meet in LDS at the end.  The token rows are loaded by every
// column tile, which is why this is for few rows.  Units are counted over the slots that have rows; in the 128-column kernel's grid
// every slot without rows is a column of workgroups that look at the tables and leave.
// Measured, 37 tokens on 22 of 128 experts, 768 x 3072 (first, second product, in a layer): 24.6, 33.7 -> 25, 22 us, the layer 71 -> 58 us.
#pragma once
#include "ffn_share.h"
#include "gemm_bf16.h"

namespace moe {

constexpr int FEW_BM = 32, FEW_BN = 32;
constexpr int FEW_D = 12, FEW_BURST = 4;             // steps in flight, steps requested together
constexpr int FEW_PER = 4;                           // slots per thread at most

struct FewItem {
    int expert, row_begin, row_end, column, reuse;
};

// The unit of this workgroup: row tiles of the slots that have rows, in slot order, the column tiles of a row tile side by side,
// cut into 8 contiguous ranges, one per XCD.  Found by the whole workgroup: every load goes out at once (the tables hold
// max_slots entries, so none has to wait for n_slots), a scan gives everybody's place, the owner of the unit writes it out.
// Returns false (for all threads) if there is nothing to do.
__device__ __forceinline__ bool few_rows_find(const int32_t *__restrict__ slot_offset,
                                              const int32_t *__restrict__ slot_expert,
                                              const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int E,
                                              int n_nt, int max_rows, FewItem &it)
{
    __shared__ int wave_sums[SHARE_THREADS / WAVE];
    __shared__ FewItem found;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int per = (max_slots + SHARE_THREADS - 1) / SHARE_THREADS;         // 1 .. FEW_PER
    const int p0 = tid * per;
    int e[FEW_PER + 2], off[FEW_PER + 1];            // slots p0 - 1 .. p0 + per, first rows of p0 .. p0 + per
    const int P = n_slots_p[0];
#pragma unroll
    for (int i = 0; i < FEW_PER + 2; ++i) {
        const int p = p0 - 1 + i;
        e[i] = i < per + 2 && p >= 0 && p < max_slots ? slot_expert[p] : -1;
    }
#pragma unroll
    for (int i = 0; i < FEW_PER + 1; ++i) off[i] = i <= per && p0 + i <= max_slots ? slot_offset[p0 + i] : 0;
    if (tid == 0) found.expert = -1;                 // stays so if the slot tables contradict themselves
    int tiles[FEW_PER], count = 0;
#pragma unroll
    for (int i = 0; i < FEW_PER; ++i) {
        const int p = p0 + i, n = (off[i + 1] < max_rows ? off[i + 1] : max_rows) - off[i];     // the grid is sized for max_rows
        const bool in = i < per && p < P && p < max_slots && e[i + 1] >= 0 && e[i + 1] < E;    // never index weights with a bad id
        // the experts schedule: one unit per expert, its first slot's, whether or not there are rows
        tiles[i] = !in ? 0 : schedule == MOE_SCHEDULE_EXPERTS ? (e[i] != e[i + 1] ? 1 : 0) : n > 0 ? (n + FEW_BM - 1) / FEW_BM : 0;
        count += tiles[i];
    }
    int inc = count;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
    }
    if (lane == 63) wave_sums[w] = inc;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int i = 0; i < SHARE_THREADS / WAVE; ++i) {
        base += i < w ? wave_sums[i] : 0;
        total += wave_sums[i];
    }
    const int lid = xcd_remap(blockIdx.x, total * n_nt);
    if (lid < 0) return false;                       // uniform
    const int item = lid / n_nt;
    int at = base + inc - count;
#pragma unroll
    for (int i = 0; i < FEW_PER; ++i) {
        if (item >= at && item < at + tiles[i]) {
            int end = off[i + 1];
            if (schedule == MOE_SCHEDULE_EXPERTS) {
                int last = p0 + i;
                while (last + 1 < P && last + 1 < max_slots && slot_expert[last + 1] == e[i + 1]) ++last;
                end = slot_offset[last + 1];
            }
            const int r0 = off[i] + (item - at) * FEW_BM;
            found.expert = e[i + 1];
            found.column = lid - item * n_nt;
            found.row_begin = r0;
            found.row_end = schedule == MOE_SCHEDULE_EXPERTS || end - r0 < FEW_BM ? end : r0 + FEW_BM;
            found.reuse = end - off[i] > FEW_BM || e[i] == e[i + 1] || e[i + 2] == e[i + 1];
        }
        at += tiles[i];
    }
    __syncthreads();
    it = found;
    return it.expert >= 0 && it.expert < E && it.row_begin >= 0;             // uniform; never index with a bad table
}

template <bool STREAM>
__device__ __forceinline__ void few_rows_tile(const bf16_t *a_row, const bf16_t *__restrict__ strip, int K,
                                              float (*__restrict__ part)[FEW_BN + 4])
{
    typedef unsigned u32x4f_t __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int steps = K / 64;                        // of 16 k, per wavefront
    const bf16_t *a = a_row + w * (K / 4) + (lane >> 5) * 8;
    const u32x4f_t *b = reinterpret_cast<const u32x4f_t *>(strip) + (size_t)w * steps * 64;      // scalar
    u32x4f_t af[FEW_D], bf[FEW_D];
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    // every load is unconditional (past the end: a harmless re-read), so that the waits can be counts
    auto load = [&](int s0, int j0) {
#pragma unroll
        for (int j = 0; j < FEW_BURST; ++j) {
            const int s = s0 + j < steps ? s0 + j : steps - 1;
            const u32x4f_t *p = b + (size_t)s * 64 + lane;
            bf[j0 + j] = STREAM ? __builtin_nontemporal_load(p) : *p;
        }
#pragma unroll
        for (int j = 0; j < FEW_BURST; ++j) {
            const int s = s0 + j < steps ? s0 + j : steps - 1;
            af[j0 + j] = *reinterpret_cast<const u32x4f_t *>(a + s * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int j) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[j]), __builtin_bit_cast(bf16x8_t, bf[j]),
                                                      acc, 0, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < FEW_D; j += FEW_BURST) load(j, j);
    int s = 0;
    for (; s + FEW_D < steps; s += FEW_D) {
#pragma unroll
        for (int j0 = 0; j0 < FEW_D; j0 += FEW_BURST) {
#pragma unroll
            for (int j = 0; j < FEW_BURST; ++j) multiply(j0 + j);
            __builtin_amdgcn_sched_barrier(0);
            load(s + FEW_D + j0, j0);
        }
    }
#pragma unroll
    for (int j = 0; j < FEW_D; ++j)
        if (s + j < steps) multiply(j);              // uniform
#pragma unroll
    for (int v = 0; v < 16; ++v) part[acc_row(v, lane)][lane & 31] = acc[v];
}

template <bool RELU>
__global__ __launch_bounds__(SHARE_THREADS, 3) void ffn_few_rows_bf16_kernel(
    const bf16_t *__restrict__ A, const bf16_t *__restrict__ Wp, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int max_rows, bf16_t *__restrict__ C)
{
    __shared__ __attribute__((aligned(16))) float part[4][FEW_BM][FEW_BN + 4];
    FewItem it;
    if (!few_rows_find(slot_offset, slot_expert, n_slots_p, max_slots, schedule, E, N / FEW_BN, max_rows, it)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const bf16_t *strip = Wp + (size_t)it.expert * K * N + (size_t)it.column * FEW_BN * K;
    const int row_end = it.row_end < max_rows ? it.row_end : max_rows;
    for (int r0 = it.row_begin; r0 < row_end; r0 += FEW_BM) {
        const int nrows = row_end - r0 < FEW_BM ? row_end - r0 : FEW_BM;
        int src = r0 + ((lane & 31) < nrows ? (lane & 31) : nrows - 1);      // rows past the tile repeat its last row
        if (row_index) {
            src = row_index[src];
            src = src >= 0 && src < n_src_rows ? src : 0;                    // a bad index reads row 0
        }
        const bf16_t *a_row = A + (size_t)src * K;
        if (it.reuse) few_rows_tile<false>(a_row, strip, K, part[w]);
        else few_rows_tile<true>(a_row, strip, K, part[w]);
        __syncthreads();
        const int r = tid >> 3, c = (tid & 7) * 4;
        if (r < nrows) {
            float o[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v = (part[0][r][c + i] + part[1][r][c + i]) + (part[2][r][c + i] + part[3][r][c + i]);
                o[i] = RELU ? (v > 0.f ? v : 0.f) : v;
            }
            *reinterpret_cast<uint2 *>(C + (size_t)(r0 + r) * N + it.column * FEW_BN + c) =
                make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
        }
        __syncthreads();
    }
}

// Where this kernel is the faster one (first / second product in us against the 128-column kernel):
//  - at most half of the slots can have a row: most of the 128-column kernel's grid is slots without rows (37 rows in 144 slots, 768 x
//    3072: 26.8 / 24.0 against 36.0 / 36.3; with rows in every slot, 36 in 36: 35 / 30 against 28 / 27);
//  - a long k and tiles for half of the CUs at most, slots of 32 rows at most on average (9 slots of 8 rows, k = 3072: 12.6 against 20.4, of
//    30 rows: 15.9 against 21.6; 8 slots of 20 rows, k = 1024: 8.5 against 9.8, k = 256: 7.6 against 6.9; 216 tiles: 14.8 against 11.4).
static inline bool ffn_few_rows(int max_rows, int max_slots, int K, int N)
{
    if (max_slots > FEW_PER * SHARE_THREADS) return false;
    if (2LL * max_rows <= max_slots) return true;
    const long long active = max_rows < max_slots ? max_rows : max_slots;
    return K >= 1024 && active * (N / 128) <= 128 && (long long)max_rows <= 32LL * max_slots;
}

// one row tile per slot that can have rows, and one per 32 rows
static inline int few_rows_grid(int max_rows, int max_slots, int schedule, int N)
{
    const int active = max_rows < max_slots ? max_rows : max_slots;
    const int items = schedule == MOE_SCHEDULE_SLOTS ? active + max_rows / FEW_BM : max_slots;
    return (int)align_up((size_t)items * (N / FEW_BN), 8);
}

}  // namespace moe
