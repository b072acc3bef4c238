// How a grouped product deals its (expert, row tile, column tile) units to workgroups without a list kernel.
#pragma once
#include "common.h"

namespace moe {

constexpr int SHARE_THREADS = 256;
constexpr int TILE_COST_TILE = 3, TILE_COST_BLOCK = 2;

// Rows of one expert (a tile of them, or in the experts schedule all) x one column tile.
struct TileItem {
    int expert, row_begin, row_end, column, reuse;
};

// A layer's last step, made by its second product (top-1 routing): what moe_combine does, row by row as the rows come out.
// The tables are those of the same batch: perm[row] is the token of a row, inv[token] < 0 a token without one.
struct LayerOut {
    const int32_t *perm, *inv;
    const float *prob;
    const void *x;
    void *out;
    int T, residual;

    // a 16-byte piece of bf16: y scaled, on x or on zero
    __device__ __forceinline__ static uint4 scaled(uint4 y, float p, uint4 base)
    {
        auto two = [&](uint32_t v, uint32_t b) {
            return pack_bf16x2(fmaf(p, __uint_as_float(v << 16), __uint_as_float(b << 16)),
                               fmaf(p, __uint_as_float(v & 0xffff0000u), __uint_as_float(b & 0xffff0000u)));
        };
        return make_uint4(two(y.x, base.x), two(y.y, base.y), two(y.z, base.z), two(y.w, base.w));
    }
    // The tokens without a row, out <- x, dealt to all wavefronts of the launch.  Where capacity drops most tokens they are many, and every trip to
    // memory stands in front of the product: a wavefront takes as many rows side by side as its lanes hold, AHEAD such passes at a time.
    // Captured layers, us, with moe_combine, a row at a time, so: fp32 64 -> 256, 4 experts, 40 of 2048 rows kept 20.8, 21.9, 19.9, 448 kept 26.8,
    // 28.0, 25.6; bf16 128 -> 256, 24 experts, 24 of 1500 kept 18.5, 19.1, 17.7.
    static constexpr int AHEAD = 4;
    struct Deal {
        int row[AHEAD];                // inv of this lane's tokens in the first passes
    };
    template <class F>
    __device__ __forceinline__ void dealt(int vec_per_row, F &&f) const
    {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));              // a copy of its own: what comes of it is not kept through the product
        const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
        const unsigned wave = blockIdx.x * (SHARE_THREADS / WAVE) + w, waves = gridDim.x * (SHARE_THREADS / WAVE);
        const int sh = vec_per_row < WAVE ? 31 - __builtin_clz(2 * vec_per_row - 1) : 6, rows = WAVE >> sh;      // 2^sh lanes per row, rows per pass
        // (T is some thousands at most: a product with it fits)
        const int token = wave < (unsigned)T ? (int)wave * rows + (lane >> sh) : T, step = (int)(waves < (unsigned)T ? waves : T) * rows;
        f(token, step, lane & ((1 << sh) - 1), 1 << sh);
    }
    __device__ __forceinline__ void ask(Deal &deal, int token, int step) const
    {
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) deal.row[p] = token + p * step < T ? inv[token + p * step] : 0;
    }
    // asked for before the search of the units, so that the answer comes with the slot tables
    __device__ __forceinline__ Deal deal_dropped(int vec_per_row) const
    {
        Deal deal;
        dealt(vec_per_row, [&](int token, int step, int, int) { ask(deal, token, step); });
        return deal;
    }
    __device__ __forceinline__ void copy_dropped(Deal deal, int vec_per_row) const
    {
        typedef unsigned vec_t __attribute__((ext_vector_type(4)));
        dealt(vec_per_row, [&](int token, int step, int piece, int lanes) {
            while (token < T) {
                int none = 0;                          // negative: one of them has no row
#pragma unroll
                for (int p = 0; p < AHEAD; ++p) none |= deal.row[p];
                for (int c = none < 0 ? piece : vec_per_row; c < vec_per_row; c += lanes) {
                    vec_t v[AHEAD];
#pragma unroll
                    for (int p = 0; p < AHEAD; ++p)
                        if (deal.row[p] < 0) v[p] = static_cast<const vec_t *>(x)[(size_t)(token + p * step) * vec_per_row + c];
#pragma unroll
                    for (int p = 0; p < AHEAD; ++p)
                        if (deal.row[p] < 0) static_cast<vec_t *>(out)[(size_t)(token + p * step) * vec_per_row + c] = v[p];
                }
                token += AHEAD * step;
                ask(deal, token, step);
            }
        });
    }
};

// Relative cost of a row tile: its 16-row blocks, and what every tile pays for its weights.
__device__ __forceinline__ int tile_cost(int rows) { return TILE_COST_TILE + TILE_COST_BLOCK * ((rows + 15) >> 4); }

// Which (expert, row tile, column tile) a workgroup works on, found from the slot tables by the whole workgroup: each
// thread counts the tiles of its slots, a scan gives everybody's place, and the owner of the tile wanted writes it out.  (A list
// built by a kernel of its own costs a launch of 4-5 us in front of the first product.)
// The slots of an expert are neighbours and so are their rows: tiles are cut over all rows of the expert (the results are the
// same, and replicas leave no part-filled tiles behind).  Order: experts as in the tables, their row tiles, the column tiles of
// a row tile side by side.  The order is cut into 8 ranges of equal COST, one per XCD; ranges of equal length left the XCDs that
// drew the full tiles of the hot experts with 1.5 times the work of the others.  Each XCD's workgroups with work come first in
// the grid: two tiles on one CU take twice as long as on two, and the launch order is what spreads them.
template <int BM>
struct TileShare {
    // this thread's slots and the tiles and cost before them
    int P, E, schedule, n_nt, max_rows, p0, p1, own_rows, count, count_base;
    int first, end;                               // units of this workgroup's XCD
    bool own;                                     // one slot per thread: expert and first row are its own
    int own_expert, own_row;

    // rows of the expert whose first slot p is, 0 for its other slots; tables that go on past max_rows end there (the grid is
    // sized for max_rows: units of the rows past it would push others out)
    __device__ __forceinline__ int rows_of(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                           int p) const
    {
        const int e = slot_expert[p];
        if (e < 0 || e >= E) return 0;            // never index weights with a bad id
        if (p > 0 && slot_expert[p - 1] == e) return 0;
        int last = p;
        while (last + 1 < P && slot_expert[last + 1] == e) ++last;
        const int r0 = slot_offset[p];
        if (r0 < 0) return 0;                     // nor go through rows that are none
        const int left = max_rows - r0;
        int n = slot_offset[last + 1] - r0;
        if (n > left) n = left;
        return n > 0 ? n : 0;
    }
    // the experts schedule makes one tile of all rows (they queue), the slot schedule tiles of BM rows
    __device__ __forceinline__ int tiles_of(int n) const
    {
        return schedule == MOE_SCHEDULE_EXPERTS ? (n > 0 ? 1 : 0) : (n + BM - 1) / BM;
    }
    __device__ __forceinline__ int full_cost() const
    {
        return schedule == MOE_SCHEDULE_EXPERTS ? TILE_COST_TILE : tile_cost(BM);
    }
    __device__ __forceinline__ int cost_of(int n, int tiles) const
    {
        if (tiles == 0) return 0;
        return schedule == MOE_SCHEDULE_EXPERTS ? TILE_COST_TILE
                                                : (tiles - 1) * tile_cost(BM) + tile_cost(n - (tiles - 1) * BM);
    }
    __device__ __forceinline__ int rows_at(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                           int p) const
    {
        return p1 - p0 == 1 ? own_rows : rows_of(slot_offset, slot_expert, p);
    }

    __device__ __forceinline__ void find(const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
                                         const int32_t *__restrict__ n_slots_p, int max_slots, TileItem *out)
    {
        constexpr int WAVES = SHARE_THREADS / WAVE;
        __shared__ int count_sums[WAVES], cost_sums[WAVES];
        __shared__ int edge_unit[2];              // first unit of this share and of the next one
        __shared__ int off_lds[SHARE_THREADS + 1];
        __shared__ unsigned long long last_lds[WAVES];
        const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
        own = max_slots <= SHARE_THREADS;             // uniform
        P = n_slots_p[0];
        int cost = 0;
        count = 0;
        if (own) {
            // A slot per thread.  Every entry is asked for at once (the tables hold max_slots entries, so none has to wait for n_slots);
            // where an expert's slots end comes from a bit per slot.  One memory round trip; walking the slots is one per slot.
            const int q = tid < max_slots ? tid : max_slots - 1;
            own_expert = slot_expert[q];
            const int before = slot_expert[q > 0 ? q - 1 : 0], after = slot_expert[q + 1 < max_slots ? q + 1 : q];
            own_row = slot_offset[q];
            const int last_row = slot_offset[max_slots];
            if (P > max_slots) P = max_slots;
            const unsigned long long ends = __ballot(tid + 1 >= P || own_expert != after);
            if (lane == 0) last_lds[w] = ends;
            if (tid < max_slots) off_lds[tid] = own_row;
            if (tid == 0) off_lds[max_slots] = last_row;
            __syncthreads();
            p0 = tid < P ? tid : P;
            p1 = tid < P ? tid + 1 : P;
            own_rows = 0;
            if (tid < P && own_expert >= 0 && own_expert < E && own_row >= 0 && (tid == 0 || before != own_expert)) {
                unsigned long long m = ends & (~0ull << lane);
                int word = w;
                while (m == 0) m = last_lds[++word];  // ends: the bit of slot P - 1 is set
                const int left = max_rows - own_row, n = off_lds[word * WAVE + __builtin_ctzll(m) + 1] - own_row;
                own_rows = n < left ? (n > 0 ? n : 0) : (left > 0 ? left : 0);
            }
            count = tiles_of(own_rows);
            cost = cost_of(own_rows, count);
        } else {
            if (P > max_slots) P = max_slots;
            const int per = (P + SHARE_THREADS - 1) / SHARE_THREADS;
            p0 = tid * per < P ? tid * per : P;
            p1 = p0 + per < P ? p0 + per : P;
            own_rows = p1 - p0 == 1 ? rows_of(slot_offset, slot_expert, p0) : 0;
            for (int p = p0; p < p1; ++p) {
                const int n = rows_at(slot_offset, slot_expert, p), t = tiles_of(n);
                count += t;
                cost += cost_of(n, t);
            }
        }
        const int count_inc = wave_scan_incl(count), cost_inc = wave_scan_incl(cost);
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
        if (tid == 0) out->expert = -1;               // stays so if the slot tables contradict themselves
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const long long edge = axis * (xcd + q) / 8;
            if (tid == 0 && edge >= axis) edge_unit[q] = n_items * n_nt;
            if (edge < axis && edge >= lo && edge < hi && own) {
                const int in = (int)(edge - lo), full = full_cost() * n_nt;
                const int tile = in / full < count - 1 ? in / full : count - 1;
                const int last = cost - (count - 1) * full_cost(), each = tile < count - 1 ? full_cost() : last;
                edge_unit[q] = (count_base + tile) * n_nt + (in - tile * full + each - 1) / each;
            } else if (edge < axis && edge >= lo && edge < hi) {
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
                                               int unit, TileItem *out) const
    {
        if (unit < count_base * n_nt || unit >= (count_base + count) * n_nt) return;
        if (own) {
            const int in = unit - count_base * n_nt, tile = in / n_nt;
            out->expert = own_expert;
            out->column = in - tile * n_nt;
            out->row_begin = own_row + tile * BM;
            out->row_end = tile + 1 < count ? own_row + (tile + 1) * BM : own_row + own_rows;
            out->reuse = own_rows > BM;
            return;
        }
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

// Workgroups enough for the XCD range with the most units: a range is an eighth of the cost, every expert has one cheap tile at
// most (its last, of one block or more), all others are full.  (With every unit counted as the cheapest, grids of long batches
// were twice as large, and went past the launch limit of 2^32 threads at half the batch.)
static inline int share_grid(int bm, int bn, int max_rows, int max_slots, int schedule, int N)
{
    long long cost = (long long)TILE_COST_TILE * max_slots, least = TILE_COST_TILE, full = TILE_COST_TILE;
    if (schedule == MOE_SCHEDULE_SLOTS) {
        cost = TILE_COST_TILE * (max_slots + (long long)max_rows / bm) + TILE_COST_BLOCK * (max_slots + (long long)max_rows / 16);
        least = TILE_COST_TILE + TILE_COST_BLOCK;
        full = TILE_COST_TILE + TILE_COST_BLOCK * (bm / 16);
    }
    const long long n_nt = N / bn, range = (cost * n_nt + 7) / 8;
    const long long last = range / least < max_slots * n_nt ? range / least : max_slots * n_nt;
    return (int)(8 * (last + (range - last * least) / full + 2));
}

}  // namespace moe
