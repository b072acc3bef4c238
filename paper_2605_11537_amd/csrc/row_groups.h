// How a kernel that gives each row to a group of lanes is launched: host rules.
#pragma once
#include "common.h"

namespace moe {

constexpr int ROW_THREADS = 256;       // threads per workgroup

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
