// binary32 grouped product of the expert FFN on the matrix cores: up to 64 rows of one slot x 64 columns per workgroup.
//
// v_mfma_f32_16x16x4_f32 multiplies and accumulates in binary32.  The four wavefronts split k, so the k loop has no LDS and
// no barrier: every wavefront streams its quarter of the rows and of the weights straight into registers, U steps of 16 k
// ahead, and the four partial tiles meet in LDS once at the end.
//   tokens   lane (g, c) of 4 x 16 loads 4 consecutive k (4g .. 4g+3) of row c: one k per instruction
//   weights  row-major as the caller keeps them: the lane loads columns 4c .. 4c+3 of each of its 4 k; column 4c + s is
//            column c of instruction strip s, so the 64 columns of the tile are 4 strips and every load is a 256-byte run
// 16-row blocks keep the padding of short slots small; blocks a tile does not have are not compiled into its body.
//
// Bound: at 47 rows per expert (1500 x 512 x 2048, 32 experts) the 134 MB of weights per product take 22 us at 6.2 TB/s and
// the padded matrix work about as long at 150 TFLOP/s; measured 64 and 91 us per product (first, second) against 77 and 130 us for a
// 64 x 64 tile on the vector units with both operands in LDS and one workgroup's whole k in one chain.
#pragma once
#include "common.h"

namespace moe {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int F32_THREADS = 256;
constexpr int F32_BM = 64, F32_BN = 64;
constexpr int F32_LD = F32_BN + 4;

// One row tile of a slot (or, in the experts schedule, all rows of an expert).
struct F32Item {
    int expert, row_begin, row_end, reuse;
};

// The tile of workgroup `bid`, found from the slot tables by the whole workgroup: each thread counts the tiles of its
// slots, a scan gives the total and the owner of the tile wanted.  A list built by a kernel of its own costs a launch of 4-5 us in
// front of the first product; this costs every workgroup about 1 us.  Tiles are dealt in 8 contiguous ranges, one per XCD,
// column tiles of a row tile side by side.
__device__ __forceinline__ bool f32_find_tile(const int32_t *__restrict__ slot_offset,
                                              const int32_t *__restrict__ slot_expert,
                                              const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int E,
                                              int n_nt, F32Item &it, int &nt)
{
    __shared__ int wave_sums[F32_THREADS / WAVE];
    __shared__ F32Item found;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int P = n_slots_p[0];
    if (P > max_slots) P = max_slots;
    const int per = (P + F32_THREADS - 1) / F32_THREADS;
    const int p0 = tid * per < P ? tid * per : P, p1 = p0 + per < P ? p0 + per : P;
    auto tiles_of = [&](int p) {
        const int e = slot_expert[p];
        if (e < 0 || e >= E) return 0;                           // never index weights with a bad id
        if (schedule == MOE_SCHEDULE_EXPERTS) return p == 0 || slot_expert[p - 1] != e ? 1 : 0;
        const int n = slot_offset[p + 1] - slot_offset[p];
        return n > 0 ? (n + F32_BM - 1) / F32_BM : 0;
    };
    int mine = 0;
    for (int p = p0; p < p1; ++p) mine += tiles_of(p);
    int inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(inc, o, 64);
        if (lane >= o) inc += v;
    }
    if (lane == 63) wave_sums[w] = inc;
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int i = 0; i < F32_THREADS / WAVE; ++i) {
        base += i < w ? wave_sums[i] : 0;
        total += wave_sums[i];
    }
    const int lid = xcd_remap(blockIdx.x, total * n_nt);
    if (lid < 0) return false;                                   // uniform
    const int item = lid / n_nt;
    nt = lid - item * n_nt;
    int at = base + inc - mine;
    if (item >= at && item < at + mine) {
        for (int p = p0; p < p1; ++p) {
            const int n = tiles_of(p);
            if (item < at + n) {
                const int e = slot_expert[p];
                int last = p;
                if (schedule == MOE_SCHEDULE_EXPERTS)
                    while (last + 1 < P && slot_expert[last + 1] == e) ++last;
                const int r0 = slot_offset[p] + (item - at) * F32_BM, end = slot_offset[last + 1];
                found.expert = e;
                found.row_begin = r0;
                found.row_end = schedule == MOE_SCHEDULE_EXPERTS || end - r0 < F32_BM ? end : r0 + F32_BM;
                found.reuse = n > 1 || end - r0 > F32_BM || (p > 0 && slot_expert[p - 1] == e) ||
                              (last + 1 < P && slot_expert[last + 1] == e);
                break;
            }
            at += n;
        }
    }
    __syncthreads();
    it = found;
    return true;
}

// part[w] <- this wavefront's share of k of (16 * MB rows) x 64 columns
template <int MB, bool STREAM>
__device__ __forceinline__ void f32_tile(const float *const (&a_row)[4], const float *__restrict__ B, int K, int N,
                                         float (*__restrict__ part)[F32_LD])
{
    constexpr int U = MB <= 2 ? 3 : 2;                           // steps of 16 k per register buffer
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, g = lane >> 4;
    const int steps = K / 64;                                    // per wavefront
    const int k_wave = w * (K / 4);                              // scalar, as are the weight rows' addresses
    const unsigned b_lane = (unsigned)(4 * g) * N + 4 * c;
    const float *a_src[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) a_src[m] = a_row[m] + k_wave + 4 * g;
    f32x4_t a[2][U][MB], b[2][U][4], acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[m][s] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    auto load = [&](int s0, int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u < steps ? s0 + u : steps - 1;   // past the end: a harmless re-read
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const f32x4_t *p = reinterpret_cast<const f32x4_t *>(B + (size_t)(k_wave + s * 16 + i) * N + b_lane);
                b[buf][u][i] = STREAM ? __builtin_nontemporal_load(p) : *p;
            }
#pragma unroll
            for (int m = 0; m < MB; ++m) a[buf][u][m] = *reinterpret_cast<const f32x4_t *>(a_src[m] + s * 16);
        }
    };
    auto multiply = [&](int s0, int buf) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u >= steps) break;                          // uniform
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int m = 0; m < MB; ++m)
#pragma unroll
                    for (int s = 0; s < 4; ++s)
                        acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[buf][u][m][i], b[buf][u][i][s], acc[m][s], 0, 0, 0);
        }
    };
    load(0, 0);
    for (int s = 0; s < steps; s += 2 * U) {
        if (s + U < steps) load(s + U, 1);
        __builtin_amdgcn_sched_barrier(0);                       // the loads stay ahead of the matrix instructions
        multiply(s, 0);
        if (s + 2 * U < steps) load(s + 2 * U, 0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(s + U, 1);
    }
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i)                              // accumulator register i: row 4g + i, column c of strip s
            *reinterpret_cast<f32x4_t *>(&part[m * 16 + 4 * g + i][4 * c]) =
                (f32x4_t){acc[m][0][i], acc[m][1][i], acc[m][2][i], acc[m][3][i]};
}

template <bool RELU>
__global__ __launch_bounds__(F32_THREADS, 2) void ffn_gemm_f32_kernel(
    const float *__restrict__ A, const float *__restrict__ W, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int schedule, int max_rows, float *__restrict__ C)
{
    __shared__ __attribute__((aligned(16))) float part[4][F32_BM][F32_LD];
    F32Item it;
    int nt;
    if (!f32_find_tile(slot_offset, slot_expert, n_slots_p, max_slots, schedule, E, N / F32_BN, it, nt)) return;
    if (it.row_begin < 0) return;                                // uniform; never index rows with a bad table
    const float *B = W + (size_t)it.expert * K * N + nt * F32_BN;
    const int tid = threadIdx.x, w = tid >> 6, c = tid & 15;
    const int row_end = it.row_end < max_rows ? it.row_end : max_rows;
    for (int r0 = it.row_begin; r0 < row_end; r0 += F32_BM) {
        const int nrows = row_end - r0 < F32_BM ? row_end - r0 : F32_BM;
        const float *a_row[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            int r = r0 + (m * 16 + c < nrows ? m * 16 + c : nrows - 1);      // rows past the tile repeat its last row
            if (row_index) {
                r = row_index[r];
                if (r < 0 || r >= n_src_rows) r = 0;             // a bad index reads row 0
            }
            a_row[m] = A + (size_t)r * K;
        }
        const int blocks = (nrows + 15) >> 4;
#define MOE_F32_TILE(M)                                                            \
    do {                                                                           \
        if (it.reuse) f32_tile<M, false>(a_row, B, K, N, part[w]);                 \
        else f32_tile<M, true>(a_row, B, K, N, part[w]);                           \
    } while (0)
        if (blocks == 1) MOE_F32_TILE(1);
        else if (blocks == 2) MOE_F32_TILE(2);
        else if (blocks == 3) MOE_F32_TILE(3);
        else MOE_F32_TILE(4);
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

// workgroups enough for every row tile the batch can have, rounded up to whole rounds over the XCDs
static inline int f32_grid(int max_rows, int max_slots, int schedule, int N)
{
    const int items = schedule == MOE_SCHEDULE_SLOTS ? max_slots + max_rows / F32_BM + 1 : max_slots;
    return (int)align_up((size_t)items * (N / F32_BN), 8);
}

}  // namespace moe
