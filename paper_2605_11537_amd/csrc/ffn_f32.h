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
// Bound: what a CU can load, about 55 GB/s (23 bytes per clock) beside the matrix instructions: a 32 x 64 tile loads 24 KB per
// 16 k where its matrix instructions take 1024 clocks.  Measured (first, second product; the vector-unit tile before, 64 x 64 with
// both operands in LDS and one workgroup's whole k in one chain, in brackets): 32 experts x 32 rows, 512 x 2048: 43, 32 us (62, 102);
// 40 slots of 10 .. 59 rows: 66, 75 us (83, 140); 8 experts x 512 rows, 768 x 3072: 215, 279 us (249, 287).
#pragma once
#include "common.h"

namespace moe {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int F32_THREADS = 256;
constexpr int F32_BN = 64;
constexpr int F32_LD = F32_BN + 4;
constexpr int F32_COST_TILE = 3, F32_COST_BLOCK = 2;

// Rows of one expert (a tile of them, or in the experts schedule all) x one column tile.
struct F32Item {
    int expert, row_begin, row_end, column, reuse;
};

// Relative cost of a row tile: its 16-row blocks, and what every tile pays for its weights.
__device__ __forceinline__ int f32_cost(int rows) { return F32_COST_TILE + F32_COST_BLOCK * ((rows + 15) >> 4); }

// Which (expert, row tile, column tile) a workgroup works on, found from the slot tables by the whole workgroup: each
// thread counts the tiles of its slots, a scan gives everybody's place, and the owner of the tile wanted writes it out.  (A list
// built by a kernel of its own costs a launch of 4-5 us in front of the first product.)
// The slots of an expert are neighbours and so are their rows: tiles are cut over all rows of the expert (the results are the
// same, and replicas leave no part-filled tiles behind).  Order: experts as in the tables, their row tiles, the column tiles of
// a row tile side by side.  The order is cut into 8 ranges of equal COST, one per XCD; ranges of equal length left the XCDs that
// drew the full tiles of the hot experts with 1.5 times the work of the others.  Each XCD's workgroups with work come first in
// the grid: a CU moves about 55 GB/s, so two tiles on one CU take twice as long as on two, and the launch order is what spreads them.
template <int BM>
struct F32Share {
    // this thread's slots and the tiles and cost before them
    int P, E, schedule, n_nt, p0, p1, own_rows, count, count_base;
    int first, end;                               // units of this workgroup's XCD

    // rows of the expert whose first slot p is, 0 for its other slots
    __device__ __forceinline__ int rows_of(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                           int p) const
    {
        const int e = slot_expert[p];
        if (e < 0 || e >= E) return 0;            // never index weights with a bad id
        if (p > 0 && slot_expert[p - 1] == e) return 0;
        int last = p;
        while (last + 1 < P && slot_expert[last + 1] == e) ++last;
        const int n = slot_offset[last + 1] - slot_offset[p];
        return n > 0 ? n : 0;
    }
    // the experts schedule makes one tile of all rows (they queue), the slot schedule tiles of BM rows
    __device__ __forceinline__ int tiles_of(int n) const
    {
        return schedule == MOE_SCHEDULE_EXPERTS ? (n > 0 ? 1 : 0) : (n + BM - 1) / BM;
    }
    __device__ __forceinline__ int full_cost() const
    {
        return schedule == MOE_SCHEDULE_EXPERTS ? F32_COST_TILE : f32_cost(BM);
    }
    __device__ __forceinline__ int cost_of(int n, int tiles) const
    {
        if (tiles == 0) return 0;
        return schedule == MOE_SCHEDULE_EXPERTS ? F32_COST_TILE
                                                : (tiles - 1) * f32_cost(BM) + f32_cost(n - (tiles - 1) * BM);
    }
    __device__ __forceinline__ int rows_at(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                           int p) const
    {
        return p1 - p0 == 1 ? own_rows : rows_of(slot_offset, slot_expert, p);
    }

    __device__ __forceinline__ void find(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                         const int32_t *__restrict__ n_slots_p, int max_slots)
    {
        constexpr int WAVES = F32_THREADS / WAVE;
        __shared__ int count_sums[WAVES], cost_sums[WAVES];
        __shared__ int edge_unit[2];              // first unit of this share and of the next one
        const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
        P = n_slots_p[0];
        if (P > max_slots) P = max_slots;
        const int per = (P + F32_THREADS - 1) / F32_THREADS;
        p0 = tid * per < P ? tid * per : P;
        p1 = p0 + per < P ? p0 + per : P;
        own_rows = p1 - p0 == 1 ? rows_of(slot_offset, slot_expert, p0) : 0;
        int cost = 0;
        count = 0;
        for (int p = p0; p < p1; ++p) {
            const int n = rows_at(slot_offset, slot_expert, p), t = tiles_of(n);
            count += t;
            cost += cost_of(n, t);
        }
        int count_inc = count, cost_inc = cost;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int a = __shfl_up(count_inc, o, 64), b = __shfl_up(cost_inc, o, 64);
            if (lane >= o) {
                count_inc += a;
                cost_inc += b;
            }
        }
        if (lane == 63) {
            count_sums[w] = count_inc;
            cost_sums[w] = cost_inc;
        }
        __syncthreads();
        int cost_base = 0, n_items = 0, cost_total = 0;
        count_base = 0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) {
            count_base += i < w ? count_sums[i] : 0;
            cost_base += i < w ? cost_sums[i] : 0;
            n_items += count_sums[i];
            cost_total += cost_sums[i];
        }
        count_base += count_inc - count;
        cost_base += cost_inc - cost;
        // a place on the cost axis, where every row tile stands n_nt times; a range takes the units that start inside it
        const long long axis = (long long)cost_total * n_nt, lo = (long long)cost_base * n_nt, hi = lo + (long long)cost * n_nt;
        const int xcd = blockIdx.x & 7;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const long long edge = axis * (xcd + q) / 8;
            if (tid == 0 && edge >= axis) edge_unit[q] = n_items * n_nt;
            if (edge < axis && edge >= lo && edge < hi) {
                int before = count_base;
                long long at = lo;
                for (int p = p0; p < p1; ++p) {
                    const int n = rows_at(slot_offset, slot_expert, p), t = tiles_of(n), c = cost_of(n, t);
                    if (edge < at + (long long)c * n_nt) {
                        const int in = (int)(edge - at), full = full_cost();
                        const int tile = in / (full * n_nt) < t - 1 ? in / (full * n_nt) : t - 1;
                        const int own = tile < t - 1 ? full : c - (t - 1) * full;
                        edge_unit[q] = (before + tile) * n_nt + (in - tile * full * n_nt + own - 1) / own;
                        break;
                    }
                    before += t;
                    at += (long long)c * n_nt;
                }
            }
        }
        __syncthreads();
        first = edge_unit[0];
        end = edge_unit[1];
    }

    // every thread calls it; the thread that owns the unit's expert writes it to *out (LDS)
    __device__ __forceinline__ void write_item(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                               int unit, F32Item *out) const
    {
        if (unit < count_base * n_nt || unit >= (count_base + count) * n_nt) return;
        int before = count_base;
        for (int p = p0; p < p1; ++p) {
            const int n = rows_at(slot_offset, slot_expert, p), t = tiles_of(n);
            if (unit < (before + t) * n_nt) {
                const int in = unit - before * n_nt, tile = in / n_nt, col = in - tile * n_nt, r0 = slot_offset[p];
                out->expert = slot_expert[p];
                out->column = col;
                out->row_begin = r0 + tile * BM;
                out->row_end = tile + 1 < t ? r0 + (tile + 1) * BM : r0 + n;
                out->reuse = n > BM;
                break;
            }
            before += t;
        }
    }
};

// part[w] <- this wavefront's share of k of (16 * MB rows) x 64 columns
template <int MB, bool STREAM, int BLOCKS>
__device__ __forceinline__ void f32_tile(const float *const (&a_row)[BLOCKS], const float *__restrict__ B, int K, int N,
                                         float (*__restrict__ part)[F32_LD])
{
    constexpr int D = 4;                                         // steps of 16 k in flight
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

template <bool RELU, int BM>
__global__ __launch_bounds__(F32_THREADS, BM == 32 ? 3 : 2) void ffn_gemm_f32_kernel(
    const float *__restrict__ A, const float *__restrict__ W, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int max_rows, float *__restrict__ C)
{
    __shared__ __attribute__((aligned(16))) float part[4][BM][F32_LD];
    __shared__ F32Item found;
    F32Share<BM> share;
    share.E = E;
    share.schedule = schedule;
    share.n_nt = N / F32_BN;
    share.find(slot_offset, slot_expert, n_slots_p, max_slots);
    const int tid = threadIdx.x, w = tid >> 6, c = tid & 15;
    const int unit = share.first + (int)(blockIdx.x >> 3);
    if (unit >= share.end) return;                               // uniform
    if (tid == 0) found.expert = -1;                             // stays so if the slot tables contradict themselves
    __syncthreads();
    share.write_item(slot_offset, slot_expert, unit, &found);
    __syncthreads();
    const F32Item it = found;
    if (it.expert < 0 || it.expert >= E || it.row_begin < 0) return;         // uniform; never index with a bad table
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
#define MOE_F32_TILE(M)                                                            \
    do {                                                                           \
        if (it.reuse) f32_tile<M, false>(a_row, B, K, N, part[w]);                 \
        else f32_tile<M, true>(a_row, B, K, N, part[w]);                           \
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
}

// Workgroups enough for the XCD range with the most tiles: a range is an eighth of the cost, and no tile costs less than
// one of a single block.
static inline int f32_grid(int bm, int max_rows, int max_slots, int schedule, int N)
{
    long long cost = (long long)F32_COST_TILE * max_slots, least = F32_COST_TILE;
    if (schedule == MOE_SCHEDULE_SLOTS) {
        cost = F32_COST_TILE * (max_slots + (long long)max_rows / bm) + F32_COST_BLOCK * (max_slots + (long long)max_rows / 16);
        least = F32_COST_TILE + F32_COST_BLOCK;
    }
    const int n_nt = N / F32_BN;
    return (int)(8 * ((cost * n_nt + 8 * least - 1) / (8 * least) + 1));
}

}  // namespace moe
