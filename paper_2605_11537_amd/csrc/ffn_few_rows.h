// bf16 grouped product for batches that leave most of the chip idle in the 128-column kernel: a decode step has rows for a
// few experts only, and 22 experts x 6 column tiles are 132 workgroups that each pull 786 KB, where a CU pulls about 55 GB/s from memory.
//
// Up to 32 rows of one expert x 32 columns per workgroup, the four wavefronts split k: four times as many workgroups, and
// no LDS and no barrier in the k loop.  Each wavefront streams its quarter of one 32-column strip of the packed image (1 KB of
// consecutive memory per load, already the matrix-core operand) and the token rows next to it straight into registers, 12
// steps of 16 k ahead, refilled in bursts of 4; the partial tiles meet in LDS at the end.  The token rows are loaded by every
// column tile, which is why this is for few rows.  Units are counted over the slots that have rows; in the 128-column kernel's grid
// every slot without rows is a column of workgroups that look at the tables and leave.  The experts schedule has a unit per expert, walked
// up to 128 rows at a time: k is split the same way, so that both schedules give the same bits.
// Measured, 37 tokens on 22 of 128 experts, 768 x 3072 (first, second product, in a layer): 24.6, 33.7 -> 25, 22 us, the layer 71 -> 58 us.
// Both products in the experts schedule (128-column kernel, units of 32 rows for every expert, now): 37 rows of 128 experts, 768 x
// 3072, 72, 94, 45 us; 64 rows, 256 x 1024, 17, 33, 14.
#pragma once
#include "ffn_share.h"
#include "gemm_bf16.h"

namespace moe {

constexpr int FEW_BM = 32, FEW_BN = 32;
constexpr int FEW_BURST = 4;                         // steps requested together
constexpr int FEW_PER = 4;                           // slots per thread at most
constexpr int FEW_TALL = 4;                          // row blocks per pass in the experts schedule

// The units: row tiles of the slots that have rows, in slot order, the column tiles of a row tile side by side, cut into 8 contiguous
// ranges, one per XCD.  In the experts schedule a unit holds all rows of an expert that has any.  Found by the whole workgroup: every load
// goes out at once (the tables hold max_slots entries, so none has to wait for n_slots), a scan gives everybody's place, the owner of a
// unit writes it out.
struct FewRows {
    int e[FEW_PER + 2], off[FEW_PER + 1];            // slots p0 - 1 .. p0 + per, first rows of p0 .. p0 + per
    int tiles[FEW_PER], end[FEW_PER];
    int at0, total;                                  // tiles before this thread's, and of all

    template <bool EXPERTS>
    __device__ __forceinline__ void scan(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                         const int32_t *__restrict__ n_slots_p, int max_slots, int E, int max_rows)
    {
        __shared__ int wave_sums[SHARE_THREADS / WAVE];
        const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
        const int per = (max_slots + SHARE_THREADS - 1) / SHARE_THREADS;     // 1 .. FEW_PER
        const int p0 = tid * per;
        const int P = n_slots_p[0];
        int count = 0;
#pragma unroll
        for (int i = 0; i < FEW_PER + 2; ++i) {
            const int p = p0 - 1 + i;
            e[i] = i < per + 2 && p >= 0 && p < max_slots ? slot_expert[p] : -1;
        }
#pragma unroll
        for (int i = 0; i < FEW_PER + 1; ++i) off[i] = i <= per && p0 + i <= max_slots ? slot_offset[p0 + i] : 0;
#pragma unroll
        for (int i = 0; i < FEW_PER; ++i) {
            const int p = p0 + i;
            const bool in = i < per && p < P && p < max_slots && e[i + 1] >= 0 && e[i + 1] < E && off[i] >= 0;   // never index with a bad table
            end[i] = off[i + 1];
            if (EXPERTS && in && e[i] != e[i + 1] && e[i + 2] == e[i + 1]) { // the expert's other slots
                int last = p;
                while (last + 1 < P && last + 1 < max_slots && slot_expert[last + 1] == e[i + 1]) ++last;
                end[i] = slot_offset[last + 1];
            }
            end[i] = end[i] < max_rows ? end[i] : max_rows;                  // the grid is sized for max_rows
            const int n = in && !(EXPERTS && e[i] == e[i + 1]) ? end[i] - off[i] : 0;
            tiles[i] = n <= 0 ? 0 : EXPERTS ? 1 : (n + FEW_BM - 1) / FEW_BM;
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
        at0 = inc - count;
        total = 0;
#pragma unroll
        for (int i = 0; i < SHARE_THREADS / WAVE; ++i) {
            at0 += i < w ? wave_sums[i] : 0;
            total += wave_sums[i];
        }
    }

    // every thread calls it; the thread that owns the row tile writes it to *out (LDS)
    template <bool EXPERTS>
    __device__ __forceinline__ void write_item(int item, int column, TileItem *out) const
    {
        int at = at0;
#pragma unroll
        for (int i = 0; i < FEW_PER; ++i) {
            if (item >= at && item < at + tiles[i]) {
                const int r0 = off[i] + (item - at) * FEW_BM;
                out->expert = e[i + 1];
                out->column = column;
                out->row_begin = r0;
                out->row_end = EXPERTS || end[i] - r0 < FEW_BM ? end[i] : r0 + FEW_BM;
                out->reuse = EXPERTS ? end[i] - off[i] > FEW_TALL * FEW_BM
                                     : end[i] - off[i] > FEW_BM || e[i] == e[i + 1] || e[i + 2] == e[i + 1];
            }
            at += tiles[i];
        }
    }
};

// part <- this wavefront's share of k of (32 * MB rows) x 32 columns
template <int MB, bool STREAM>
__device__ __forceinline__ void few_rows_tile(const bf16_t *const (&a_row)[MB], const bf16_t *__restrict__ strip, int K,
                                              float (*__restrict__ part)[FEW_BN + 4])
{
    typedef unsigned u32x4f_t __attribute__((ext_vector_type(4)));
    constexpr int D = MB > 2 ? 4 : MB > 1 ? 8 : 12;  // steps in flight
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int steps = K / 64;                        // of 16 k, per wavefront
    const bf16_t *a[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) a[m] = a_row[m] + w * (K / 4) + (lane >> 5) * 8;
    const u32x4f_t *b = reinterpret_cast<const u32x4f_t *>(strip) + (size_t)w * steps * 64;      // scalar
    u32x4f_t af[D][MB], bf[D];
    f32x16_t acc[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[m][v] = 0.f;
    // Every load of a burst is unconditional, so that the waits can be counts.  k is a multiple of 128, the steps are even in number:
    // a burst that reaches past the end re-reads its last pair.
    static_assert(FEW_BURST == 4, "two pairs");
    auto load = [&](int s0, int j0) {
        const int s1 = s0 + 2 < steps ? s0 + 2 : steps - 2;
#pragma unroll
        for (int j = 0; j < FEW_BURST; ++j) {
            const u32x4f_t *p = b + (size_t)(j < 2 ? s0 : s1) * 64 + (j & 1) * 64 + lane;
            bf[j0 + j] = STREAM ? __builtin_nontemporal_load(p) : *p;
        }
#pragma unroll
        for (int j = 0; j < FEW_BURST; ++j)
#pragma unroll
            for (int m = 0; m < MB; ++m)
                af[j0 + j][m] = *reinterpret_cast<const u32x4f_t *>(a[m] + (j < 2 ? s0 : s1) * 16 + (j & 1) * 16);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int j) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
            acc[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af[j][m]),
                                                             __builtin_bit_cast(bf16x8_t, bf[j]), acc[m], 0, 0, 0);
    };
    // The bursts that a short or ragged k does not have are left out (uniform): asked for, they were two thirds of the loads of k = 256.
    // The rounds before the last stay unconditional.
    int s = 0;
    if (steps >= D) {
#pragma unroll
        for (int j = 0; j < D; j += FEW_BURST) load(j, j);
        for (; s + 2 * D <= steps; s += D) {
#pragma unroll
            for (int j0 = 0; j0 < D; j0 += FEW_BURST) {
#pragma unroll
                for (int j = 0; j < FEW_BURST; ++j) multiply(j0 + j);
                __builtin_amdgcn_sched_barrier(0);
                load(s + D + j0, j0);
            }
        }
        if (s + D < steps) {
#pragma unroll
            for (int j0 = 0; j0 < D; j0 += FEW_BURST) {
#pragma unroll
                for (int j = 0; j < FEW_BURST; ++j) multiply(j0 + j);
                __builtin_amdgcn_sched_barrier(0);
                if (s + D + j0 < steps) load(s + D + j0, j0);
            }
            s += D;
        }
    } else {
        asm volatile("; a short k" ::: "memory");    // keeps the common first loads in their branches
#pragma unroll
        for (int j = 0; j < D; j += FEW_BURST)
            if (j < steps) load(j, j);
    }
#pragma unroll
    for (int j = 0; j < D; ++j)
        if (s + j < steps) multiply(j);              // uniform
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int v = 0; v < 16; ++v) part[m * 32 + acc_row(v, lane)][lane & 31] = acc[m][v];
}

// EXPERTS: the experts schedule, whose units are walked FEW_TALL * 32 rows at a time (fewer where there are fewer)
template <bool RELU, bool EXPERTS>
__global__ __launch_bounds__(SHARE_THREADS, EXPERTS ? 2 : 3) void ffn_few_rows_bf16_kernel(
    const bf16_t *__restrict__ A, const bf16_t *__restrict__ Wp, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int max_rows, bf16_t *__restrict__ C)
{
    constexpr int TALL = EXPERTS ? FEW_TALL : 1, BM = TALL * FEW_BM;
    __shared__ __attribute__((aligned(16))) float part[4][BM][FEW_BN + 4];
    __shared__ TileItem found;
    FewRows units;
    units.scan<EXPERTS>(slot_offset, slot_expert, n_slots_p, max_slots, E, max_rows);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, n_nt = N / FEW_BN;
    const int n_units = units.total * n_nt, per_xcd = (n_units + 7) >> 3;
    for (int slot = blockIdx.x >> 3; slot < per_xcd; slot += gridDim.x >> 3) {
        const int unit = (blockIdx.x & 7) * per_xcd + slot;
        if (unit >= n_units) break;                                  // uniform
        units.write_item<EXPERTS>(unit / n_nt, unit % n_nt, &found);
        __syncthreads();
        const TileItem it = found;
        const bf16_t *strip = Wp + (size_t)it.expert * K * N + (size_t)it.column * FEW_BN * K;
        const int row_end = it.row_end;                              // past row_begin: a unit has a row, so every unit ends in a barrier
        for (int r0 = it.row_begin; r0 < row_end; r0 += BM) {
            const int nrows = row_end - r0 < BM ? row_end - r0 : BM;
            auto tile = [&](auto BLOCKS) {
                constexpr int MB = decltype(BLOCKS)::value;
                const bf16_t *a_row[MB];
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int r = m * 32 + (lane & 31);
                    int src = r0 + (r < nrows ? r : nrows - 1);                  // rows past the tile repeat its last row
                    if (row_index) {
                        src = row_index[src];
                        src = src >= 0 && src < n_src_rows ? src : 0;            // a bad index reads row 0
                    }
                    a_row[m] = A + (size_t)src * K;
                }
                if (it.reuse) few_rows_tile<MB, false>(a_row, strip, K, part[w]);
                else few_rows_tile<MB, true>(a_row, strip, K, part[w]);
            };
            if (!EXPERTS || nrows <= 32) tile(std::integral_constant<int, 1>{});
            else if (nrows <= 64) tile(std::integral_constant<int, TALL < 2 ? 1 : 2>{});
            else tile(std::integral_constant<int, TALL>{});
            __syncthreads();
            const int c = (tid & 7) * 4;
            for (int r = tid >> 3; r < nrows; r += SHARE_THREADS / 8) {
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
}

// Where this kernel is the faster one:
//  - at most half of the slots can have a row: most of the 128-column kernel's grid is slots without rows.  Both products against that
//    kernel, rows dealt evenly (by Zipf's law), us: 36 rows in 144 slots, 768 x 3072: 53, 72 (44, 70), 72 rows 91, 100 (62, 93), 144
//    rows 138, 151 (96, 115); 256 x 1024, 72 rows 17, 22 (15, 21), 216 rows 28.6, 28.2 (20, 23); 300 rows in 600 slots, 256 x 1024:
//    51.6, 50.9 (30.7, 31.8).  So the line could lie at twice as many rows for wide matrices; at half it loses nothing.  Matrices of
//    under 131072 elements are latency alone: 128 x 256, 18 rows in 36 slots 7.6, 7.2, 144 in 288 9.5, 8.4.
//  - a long k and tiles for half of the CUs at most, slots of 32 rows at most on average (9 slots of 8 rows, k = 3072: 12.6 against 20.4, of
//    30 rows: 15.9 against 21.6; 8 slots of 20 rows, k = 1024: 8.5 against 9.8, k = 256: 7.6 against 6.9; 216 tiles: 14.8 against 11.4).
static inline bool ffn_few_rows(int max_rows, int max_slots, int K, int N)
{
    if (max_slots > FEW_PER * SHARE_THREADS) return false;
    if (2LL * max_rows <= max_slots && (long long)K * N >= 131072) return true;
    const long long active = max_rows < max_slots ? max_rows : max_slots;
    return K >= 1024 && active * (N / 128) <= 128 && (long long)max_rows <= 32LL * max_slots;
}

// A workgroup per unit (one row tile per slot that can have rows, and in the slot schedule one per 32 rows), up to as many as are
// resident at once (three and two per CU): a workgroup that finds nothing to do costs 2 us of its place all the same, and most of the units
// that could be there are not.
static inline int few_rows_grid(int max_rows, int max_slots, int schedule, int N)
{
    const int active = max_rows < max_slots ? max_rows : max_slots;
    const long long units = (long long)(schedule == MOE_SCHEDULE_SLOTS ? active + max_rows / FEW_BM : active) * (N / FEW_BN);
    const int resident = 256 * (schedule == MOE_SCHEDULE_SLOTS ? 3 : 2);
    return units < resident ? (int)align_up((size_t)units, 8) : resident;
}

}  // namespace moe
