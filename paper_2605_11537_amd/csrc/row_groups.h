// How a kernel that gives each row to a group of lanes is launched: host rules.
#pragma once
#include "common.h"

namespace moe {

constexpr int ROW_THREADS = 256;       // threads per workgroup

// log2 of the lanes that share a row of vec_per_row 16-byte pieces, at least as many as it has, 1024 at most (four workgroups)
static inline int row_lanes(int vec_per_row)
{
    int lg = 0;
    while (lg < 10 && (1 << lg) < vec_per_row) ++lg;
    return lg;
}

// moe_combine: log2 of the lanes per row, one piece per lane and trip; -1: 32 lanes with three pieces each.
//  - rows of up to 32 pieces: no idle lanes (32 for every row against 1 .. 16: 65536 x 8 bf16 4.9 against 2.7 us, 1048576 x 64: 76
//    against 57);
//  - few rows: one trip per row (64 x 4096: 4.3 against 2.4 us; 2048 x 1024: 3.1 against 2.9);
//  - the widest, up to 96 MiB: the same (4096 x 4096: 12.6 against 11.1 us; 64 MiB: 23.5 and 21.0; 128 MiB: 42.2 and 44.7);
//  - else 32 lanes, which read inv and prob the fewest times per piece (32768 x 4096: 89 against 105 us; 32768 x 768: 16.8, 17.4).
static inline int combine_lanes(int T, int vec_per_row)
{
    const int lg = row_lanes(vec_per_row);
    return lg <= 5 || T <= 2048 || (vec_per_row >= 512 && (size_t)T * vec_per_row * 16 < (size_t)96 << 20) ? lg : -1;
}

// moe_combine_topk: always one piece per lane and trip, since a lane holds k of each (three at a time: 8192 x 384, k = 2: 5.4
// against 4.5 us).  Rows of up to 32 pieces, few rows and the widest ones as above (65536 x 8, k = 3: 15.5 against 3.5 us; 64 x 1024, k =
// 2: 3.8 against 2.6; 32768 x 2048: 78 against 70); else 64 lanes, from 4096 rows on 32 (32768 x 384: 14.1 against 13.6 us).
static inline int combine_topk_lanes(int T, int vec_per_row)
{
    const int lg = row_lanes(vec_per_row);
    return lg <= 5 || T <= 2048 || vec_per_row >= 256 ? lg : T <= 4096 ? 6 : 5;
}

// Grid for 2^lg lanes per row: the launch limit of 2^32 threads holds per dimension, so what goes past it lies in y.  Workgroup
// number: blockIdx.y * gridDim.x + blockIdx.x (some lie past the last row).
static inline dim3 rows_grid(int rows, int lg)
{
    constexpr int LG_THREADS = 8;
    static_assert(1 << LG_THREADS == ROW_THREADS, "");
    const long long per = 1 << (lg < LG_THREADS ? LG_THREADS - lg : 0), of = 1 << (lg > LG_THREADS ? lg - LG_THREADS : 0);
    const long long n = ((long long)rows + per - 1) / per * of, x = n < (1 << 22) ? n : 1 << 22;
    return dim3((unsigned)x, (unsigned)((n + x - 1) / x));
}

}  // namespace moe
