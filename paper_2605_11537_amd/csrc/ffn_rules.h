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
// leave less of the chip idle.  Both products, us, this kernel and the 128-row LDS tiles, rows dealt evenly: 16384 rows over 16 experts, 768 x
// 3072 (192 tiles) 184, 191; 16384 over 8, 512 x 2048 (128) 96, 89; 10032 over 16, 768 x 3072 (117) 132, 112; 16384 over 8, 256 x 1024 (64) 46, 34;
// 8192 over 64, 512 x 2048 (128) 85, 80.  The line suits the rows that a plan keeps of max_rows; where it keeps all of them, or a few slots hold
// most, it lies a little high: 12288 over 8, 768 x 3072 (144), 9800 kept of a deal by Zipf's law 131, 112, all of it 141, 151, evenly 141, 148; 16384
// over 32, 512 x 2048 (128) 10600 kept 82, 77, all 101, 108, evenly 94, 89; and in narrow products by more: 40000 over 159, 256 x 1024 (159) 24000 kept
// 66, 77, all 91, 106, evenly 87, 102.  At d = 1024 half of the CUs are enough: 8192 rows over 8, 1024 x 4096 (128), by Zipf's law 170, 183, evenly
// 156, 148.
// Nor is it taken where the weight stream binds (ffn_weight_stream) and a slot is a tile of the 128-column kernel: that one keeps more weights in
// flight.  Both products, us, this kernel and that, rows kept of a deal by Zipf's law: 768 x 3072, 128 experts, 7834 of 12288 rows 323, 259; 64
// experts, 4705 of 8192 164, 137; 256 experts, 14826 of 30000 542, 521; 512 x 2048, 256 experts, 12567 of 20000 253, 218; 1024 x 4096, 32 experts,
// 2548 of 4096 158, 140.  At d = 1024 with a tile for every CU they are about even (64 experts, 8192 rows evenly 243, 252, 5000 of them kept 251,
// 233), with more than 128 rows per slot a second tile reads the weights again (64 x 140 rows: 170, 212).  From 96 tiles on this kernel is taken
// where the weights stream: 32 experts, 8192 rows, 768 x 3072 141, LDS tiles 138 -- and 126 in the 128-column kernel, for slots of two full tiles.
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
// (128 MB per product under 128 rows per slot belong to the 128-column kernel: 64 experts, 4705 of 8192 rows kept, 768 x 3072 137 us against 182,
// 128 rows each 162, 164; 512 x 2048, which these take below 64 experts, 64 x 128 79, 80, 32 x 128 50, 40).
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
//     Outputs of more than 4 MB lose where capacity drops most of the rows, which then are copied in front of the product (kept of rows: 1024 -> 4096, 16
//     experts, 336 of 1400 127.9, 133.9, 30 experts, 60 of 1322 192.3, 197.1; 768 -> 1536, 83 experts, 562 of 1592 170.1, 175.3; 256 -> 512, 32 experts, 96 of
//     6000 33.3, 33.7), and gain 1 % at most where it does not.
//   bf16, 128-column kernel: 256 -> 1024, 64 experts, 200 rows 25.9, 24.4, 1000 rows 31.8, 30.3; 512 -> 2048, 32 experts, 200 rows 40.1, 38.2; on
//     average 1.5 % up to 1000 rows over 64 .. 768 columns and more, none from 2000 on (768 -> 3072, 64 experts, 2048 rows 124.3, 125.7).  Between
//     them 2.3 % on average over 64 layers of 800 .. 1500 rows, at worst 0.9 % lost (128 -> 256, 24 experts, 1489 rows 26.6, 26.8); 1500 rows: 256 ->
//     1024, 64 experts 36.8, 35.5, 512 -> 2048, 32 experts 51.8, 49.9.  With a work list: 1024 -> 4096, 16 experts, 1024 rows 83.8, 79.6, 1500 rows
//     95.4, 92.8; 2048 -> 8192, 8 experts, 1500 rows 236.2, 237.1.
//   The others lost or gained nothing: the 128-row tiles 256 -> 1024, 8 experts, 2000 rows 32.4, 33.6; the kernel for few rows has no registers
//     left for it (37 rows, 128 experts 56.5, 57.4).
// Nor in the experts schedule, whose few workgroups write one after another (64 -> 256, 32 experts, 2048 fp32 rows 98, 105).
static inline bool ffn_output_pays(int T, int max_slots, int E, int d, int F, int dtype, int schedule)
{
    if (schedule != MOE_SCHEDULE_SLOTS || T <= 0 || max_slots <= 0 || E <= 0 || d <= 0 || F <= 0) return false;
    if (dtype == MOE_F32) return T <= (d >= 128 && d <= 256 ? 6000 : 2048) && (long long)T * d <= 1 << 20;
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
