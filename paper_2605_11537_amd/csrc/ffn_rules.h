// Which kernel takes the bf16 expert products.  Host code without a launch in it, so that a test can ask what a shape takes.
#pragma once
#include "ffn_few_rows.h"
#include "ffn_lds_tile.h"

namespace moe {

// The 256 x 256 tile pays off when slots are long: it can be launched when the rows could fill slots of
// 64 and more on average and the matrix sizes fit its tiling (and is where its tiles fill the chip, see ffn_dense_fills).
static inline bool ffn_use_dense(int max_rows, int max_slots, int K, int N, int schedule)
{
    return schedule == MOE_SCHEDULE_SLOTS && N % DENSE_BN == 0 && N <= DENSE_MAX_N && K % DENSE_BK == 0 && K >= DENSE_MIN_K &&
           (long long)max_rows >= 64LL * max_slots && max_rows >= 4096;
}

// From 128 MB of weights per product on, their stream binds at the few hundred rows per slot that these kernels see.
static inline bool ffn_weight_stream(int E, int d, int F) { return (long long)E * d * F >= (64LL << 20); }

// Tiles of the product with fewer columns that can be expected (a slot has one at least): under five eighths of the CUs the others
// leave less of the chip idle.  Both products, us, this kernel and the one taken instead: 16384 rows over 16 experts, 768 x 3072 (192 tiles) 198, 229;
// 16384 over 8, 512 x 2048 (128) 95, 85; 10032 over 16, 768 x 3072 (117) 139, 113; 16384 over 8, 256 x 1024 (64) 47, 34; 8192 over 64, 512 x 2048
// (128) 84, 78.  The line suits the rows that a plan keeps of max_rows; where it keeps all of them, or a few slots hold most, it lies a little high:
// 12288 over 8, 768 x 3072 (144), at most 1920 per expert 119, 107, evenly 142, 153; 16384 over 32, 512 x 2048 (128), at most 641 84, 77, evenly 94,
// 89, by Zipf's law 102, 113; 40000 over 159, 256 x 1024 (159) 68, 73, 87, 103, 106, 106.  At d = 1024 half of the CUs are enough: 8192 rows over 8, 1024 x 4096 (128), dealt by Zipf's law 160, 177, evenly 155, 141.
// Nor is it taken where the weight stream binds (ffn_weight_stream) and a slot is a tile of the 128-column kernel: that one keeps more weights in
// flight.  Both products, us, this kernel and that: 768 x 3072, 128 experts, 12288 rows of which a plan keeps 7834 299, 262; 64 experts,
// 8192 rows, 4705 kept 166, 141; 256 experts, 30000 rows, 14826 kept 546, 519; 512 x 2048, 256 experts, 20000 rows, 12567 kept 262, 227; 1024 x 4096,
// 32 experts, 4096 rows, 2548 kept 163, 141.  At d = 1024 with a tile for every CU they are even (64 experts, 8192 rows: 246, 238 and 245, 267),
// with more than 128 rows per slot a second tile reads the weights again (64 x 140 rows: 170, 210; 32 experts, 8192 rows, 768 x 3072, from 96 tiles
// on: 149, 158 on the LDS tiles).
static inline bool ffn_dense_fills(int max_rows, int max_slots, int E, int d, int F)
{
    const long long ranges = max_rows / DENSE_BM > max_slots ? max_rows / DENSE_BM : max_slots;
    const int n = d < F ? d : F;
    const long long tiles = ranges * (n / DENSE_BN);
    const bool stream = ffn_weight_stream(E, d, F);
    if (stream && (long long)max_rows <= 128LL * max_slots && (n < 1024 || tiles < 256)) return false;
    return tiles >= (n >= 1024 ? 128 : stream ? 96 : 160);
}

// Where the 128-row LDS tiles take the products (of batches whose slots are not all short): the slot schedule, and no weight stream that binds
// (128 MB per product under 128 rows per slot belong to the 128-column kernel: 64 experts x 128 rows, 768 x 3072, 160 us against 175;
// 512 x 2048, 64 x 128, 78 both, 32 x 128 47 against 43).
static inline bool ffn_mid(int max_rows, int max_slots, int E, int d, int F, int schedule)
{
    return schedule == MOE_SCHEDULE_SLOTS && (!ffn_weight_stream(E, d, F) || (long long)max_rows > 128LL * max_slots);
}

enum FfnKernel { FFN_COLUMNS, FFN_DENSE, FFN_LDS_TILE };       // 128-column tiles, 256 x 256 tiles, 128-row tiles through LDS
struct FfnRoute {
    FfnKernel kernel;
    bool list;                   // a work list in front
    bool few_rows[2];            // first, second product on the kernel for few rows instead of the 128-column one
};

// Both products take the 256 x 256 tiles or neither: their list splits the rows once.
// Without them (small batches, short slots on average, shapes outside their tiling, the experts schedule) the 128-column kernel
// cuts work items 128 rows high and picks the tile height per item; with them it is not launched at all.
// Slots that hold 64 rows on average at most are one tile each, give or take (unless the batch is one that the 256 x 256 kernel could
// take: its slots may be long): the 128-column kernel then reads the slot tables itself and the list kernel (a launch of ~5 us
// in front of the first product) is skipped.  Long slots keep the list: it cuts them into tiles that run side by side.
static inline FfnRoute ffn_route(int max_rows, int max_slots, int E, int d, int F, int schedule)
{
    const bool fits = ffn_use_dense(max_rows, max_slots, d, F, schedule) && ffn_use_dense(max_rows, max_slots, F, d, schedule);
    if (fits && ffn_dense_fills(max_rows, max_slots, E, d, F)) return {FFN_DENSE, true, {false, false}};
    const bool short_slots = !fits && (long long)max_rows <= 64LL * max_slots;
    if (!short_slots && ffn_mid(max_rows, max_slots, E, d, F, schedule)) return {FFN_LDS_TILE, false, {false, false}};
    return {FFN_COLUMNS, !short_slots,
            {short_slots && ffn_few_rows(max_rows, max_slots, d, F), short_slots && ffn_few_rows(max_rows, max_slots, F, d)}};
}

// Where the second product of a layer makes the output: a launch less, and y is not read back; but the rows then leave scattered from
// workgroups that still compute, which costs more than the launch where there are many.  Captured layers, us, with moe_combine and so.
//   binary32: 64 -> 256, 32 experts, 100 rows 19.7, 17.6; 256 -> 1024, 8 experts, 16 rows 22.8, 20.5, 1500 rows 58.7, 53.0, 32 experts,
//     4096 rows 75.9, 71.2; 512 -> 2048, 32 experts, 1500 rows 117, 114.  Past the lines: 64 -> 256, 8 experts, 4096 rows 29.8, 30.9; 64 -> 1024, 128
//     experts, 16384 rows 82, 85; 512 -> 2048 is even from 3000 rows on (0.98 .. 1.02).
//   bf16, 128-column kernel: 256 -> 1024, 64 experts, 200 rows 25.9, 24.4, 1000 rows 31.8, 30.3; 512 -> 2048, 32 experts, 200 rows 40.1, 38.2; on
//     average 1.5 % up to 1000 rows over 64 .. 768 columns and more, none from 2000 on (768 -> 3072, 64 experts, 2048 rows 124.3, 125.7).
//   The others lost or gained nothing: the 128-row tiles 256 -> 1024, 8 experts, 2000 rows 32.4, 33.6; the kernel for few rows has no registers
//     left for it (37 rows, 128 experts 56.5, 57.4).
// Nor in the experts schedule, whose few workgroups write one after another (64 -> 256, 32 experts, 2048 fp32 rows 98, 105).
static inline bool ffn_output_pays(int T, int max_slots, int E, int d, int F, int dtype, int schedule)
{
    if (schedule != MOE_SCHEDULE_SLOTS || T <= 0 || max_slots <= 0 || E <= 0 || d <= 0 || F <= 0) return false;
    if (dtype == MOE_F32) return T <= (d >= 128 && d <= 256 ? 6000 : 2048);
    if (dtype != MOE_BF16 || T > 1500) return false;
    const FfnRoute route = ffn_route(T, max_slots, E, d, F, schedule);
    return route.kernel == FFN_COLUMNS && !route.few_rows[1];
}

// Whether the second product of a layer can write the output: it then reads its own operands while it writes, moe_combine does not read
// them any more.  An output that lies in one of them (its caller has no more use for h, say) is made behind the product.  ws_bytes: of
// the products' workspace, the part that they use.
static inline bool ffn_output_apart(const moe_layer_args *a, int max_slots, size_t ws_bytes)
{
    const size_t esz = a->dtype == MOE_F32 ? 4 : 2, bytes = (size_t)a->T * a->d * esz;
    const uintptr_t out = reinterpret_cast<uintptr_t>(a->out);
    auto apart = [&](const void *p, size_t n) {
        const uintptr_t at = reinterpret_cast<uintptr_t>(p);
        return at >= out ? at - out >= bytes : out - at >= n;
    };
    return apart(a->ffn_ws, ws_bytes) && apart(a->w2, (size_t)a->E * a->F * a->d * esz) && apart(a->perm, (size_t)a->T * 4) &&
           apart(a->slot_offset, ((size_t)max_slots + 1) * 4) && apart(a->slot_expert, (size_t)max_slots * 4) && apart(a->n_slots, 4);
}

}  // namespace moe
