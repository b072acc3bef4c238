// moe_combine: scale expert outputs by the gate probability and scatter them back to token
// order; tokens over capacity are copied through bit for bit.  HBM-bound: every 16-byte
// piece of x, y_perm and out is touched once.
#include "route.h"
#include "row_groups.h"

namespace moe {

constexpr int CMB_THREADS = ROW_THREADS;

typedef unsigned cmb_u32x4_t __attribute__((ext_vector_type(4)));
constexpr int CMB_PIECES = 3;                            // 16-byte pieces per lane and trip

// A group of lanes per row: the row index is a shift (a 64-bit division per piece was as long as the piece's other work), inv and
// prob are read once per row, and a lane has its pieces of a trip in flight behind them.
// PIECES 3: 32 lanes.  PIECES 1: 2^lg lanes, as many as the row has pieces (combine_lanes below).
// Measured inside its callers, 65536 x 768 bf16: 41.1 -> 36.8 us, with the residual 49.6 -> 48.7 us (two rows per group of lanes:
// 39 and 52 us); without the stores past the L2s 46 us.
// STREAM: an output far beyond what the L2s (32 MiB) hold is written past them, and with the residual's second input stream y is
// read past them too.  The row copy of moe_dispatch has the same line.  What it gives and costs depends on what follows (both calls
// in turn, in bf16 rows of 768; without and with it, in brackets with a pass over x_perm between them and one over the output after):
// 48 MiB 47, 47 us (79, 82); 72 MiB 65, 58 (103, 108); 96 MiB 93, 74 (134, 142); 127 MiB 117, 98 (179, 195); 192 MiB 172, 160 (291,
// 285); 288 MiB 256, 242 (469, 456).  So the line lies where the calls themselves gain, and a reader that follows at once pays 2 .. 8 %
// of the whole for finding less in the caches, up to about 150 MiB.
constexpr size_t CMB_STREAM_BYTES = (size_t)64 << 20;

// this thread's row, its place in the row's group and the size of the group
template <int PIECES>
__device__ __forceinline__ unsigned combine_row(int lg, int &lane, int &lanes)
{
    const unsigned wg = blockIdx.y * gridDim.x + blockIdx.x;
    const int shift = PIECES > 1 ? 5 : lg;
    lanes = 1 << shift;
    if (shift > 8) {                                     // a row over several workgroups
        lane = (wg & ((lanes >> 8) - 1)) * CMB_THREADS + threadIdx.x;
        return wg >> (shift - 8);
    }
    lane = threadIdx.x & (lanes - 1);
    return wg * (CMB_THREADS >> shift) + (threadIdx.x >> shift);
}

template <bool BF16, bool RESIDUAL, bool STREAM, int PIECES>
__global__ __launch_bounds__(CMB_THREADS) void combine_kernel(const cmb_u32x4_t *__restrict__ y_perm,
                                                              const cmb_u32x4_t *__restrict__ x,
                                                              const int32_t *__restrict__ inv,
                                                              const float *__restrict__ prob, int T, int vec_per_row, int lg,
                                                              cmb_u32x4_t *__restrict__ out)
{
    int lane, lanes;
    const unsigned s = combine_row<PIECES>(lg, lane, lanes);
    if (s >= (unsigned)T) return;
    const int pos = inv[s];
    const float p = prob[s];
    const cmb_u32x4_t *xr = x + (size_t)s * vec_per_row;
    // a dropped row reads its x in place of y (and passes it through)
    const cmb_u32x4_t *yr = pos >= 0 ? y_perm + (size_t)pos * vec_per_row : xr;
    cmb_u32x4_t *o = out + (size_t)s * vec_per_row;
    for (int c0 = lane; c0 < vec_per_row; c0 += lanes * PIECES) {
        cmb_u32x4_t yv[PIECES], xv[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int c = c0 + i * lanes;
            if (c >= vec_per_row) continue;
            yv[i] = STREAM && RESIDUAL ? __builtin_nontemporal_load(yr + c) : yr[c];
            if (RESIDUAL) xv[i] = xr[c];
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int c = c0 + i * lanes;
            if (c >= vec_per_row) continue;
            cmb_u32x4_t r = yv[i];
            if (pos >= 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t y = yv[i][k], b = RESIDUAL ? xv[i][k] : 0u;
                    if (BF16)
                        r[k] = pack_bf16x2(fmaf(p, __uint_as_float(y << 16), __uint_as_float(b << 16)),
                                           fmaf(p, __uint_as_float(y & 0xffff0000u), __uint_as_float(b & 0xffff0000u)));
                    else
                        r[k] = __float_as_uint(fmaf(p, __uint_as_float(y), __uint_as_float(b)));
                }
            }
            if (STREAM) __builtin_nontemporal_store(r, o + c);
            else o[c] = r;
        }
    }
}

// top-k: k gathered rows per token, accumulated in choice order in binary32, one rounding; 2^lg lanes per row as above
template <bool BF16, bool RESIDUAL>
__global__ __launch_bounds__(CMB_THREADS) void combine_topk_kernel(const cmb_u32x4_t *__restrict__ y_perm,
                                                                   const cmb_u32x4_t *__restrict__ x,
                                                                   const int32_t *__restrict__ inv,
                                                                   const float *__restrict__ weight, int T, int k,
                                                                   int vec_per_row, int lg, cmb_u32x4_t *__restrict__ out)
{
    constexpr int V = BF16 ? 8 : 4;                      // values per piece
    int lane, lanes;
    const unsigned s = combine_row<1>(lg, lane, lanes);
    if (s >= (unsigned)T) return;
    int pos[MOE_MAX_TOPK];
    float p[MOE_MAX_TOPK];
    bool any = false;
#pragma unroll
    for (int j = 0; j < MOE_MAX_TOPK; ++j) {
        pos[j] = j < k ? inv[(size_t)j * T + s] : -1;
        p[j] = j < k ? weight[(size_t)j * T + s] : 0.f;
        any = any || pos[j] >= 0;
    }
    const cmb_u32x4_t *xr = x + (size_t)s * vec_per_row;
    cmb_u32x4_t *o = out + (size_t)s * vec_per_row;
    for (int c = lane; c < vec_per_row; c += lanes) {
        cmb_u32x4_t yv[MOE_MAX_TOPK], xv;
        if (!any || RESIDUAL) xv = xr[c];
#pragma unroll
        for (int j = 0; j < MOE_MAX_TOPK; ++j)
            if (pos[j] >= 0) yv[j] = y_perm[(size_t)pos[j] * vec_per_row + c];
        if (!any) {
            o[c] = xv;
            continue;
        }
        float acc[V];
#pragma unroll
        for (int q = 0; q < V; ++q) {
            const uint32_t b = RESIDUAL ? xv[BF16 ? q / 2 : q] : 0u;
            acc[q] = __uint_as_float(!BF16 ? b : (q & 1) ? b & 0xffff0000u : b << 16);
        }
#pragma unroll
        for (int j = 0; j < MOE_MAX_TOPK; ++j) {
            if (pos[j] < 0) continue;
#pragma unroll
            for (int q = 0; q < V; ++q) {
                const uint32_t y = yv[j][BF16 ? q / 2 : q];
                acc[q] = fmaf(p[j], __uint_as_float(!BF16 ? y : (q & 1) ? y & 0xffff0000u : y << 16), acc[q]);
            }
        }
        cmb_u32x4_t r;
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = BF16 ? pack_bf16x2(acc[(2 * q) % V], acc[(2 * q + 1) % V]) : __float_as_uint(acc[q]);
        o[c] = r;
    }
}

}  // namespace moe

using namespace moe;

int moe::combine_check(const void *y_perm, const void *x, const int32_t *inv, const float *expert_prob, int T, int d, int dtype,
                       int residual, const void *out)
{
    MOE_REQUIRE(T >= 0 && d > 0, MOE_ERR_INVALID_ARG, "moe_combine: T=%d d=%d out of range", T, d);
    MOE_REQUIRE(dtype == MOE_F32 || dtype == MOE_BF16, MOE_ERR_INVALID_ARG, "moe_combine: unknown dtype %d",
                dtype);
    MOE_REQUIRE(residual == 0 || residual == 1, MOE_ERR_INVALID_ARG, "moe_combine: residual must be 0 or 1");
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(y_perm && x && inv && expert_prob && out, MOE_ERR_INVALID_ARG, "moe_combine: null pointer");
    MOE_REQUIRE(out != x && out != y_perm, MOE_ERR_INVALID_ARG, "moe_combine: out aliases an input");
    size_t esz = dtype == MOE_F32 ? 4 : 2;
    MOE_REQUIRE(((size_t)d * esz) % 16 == 0, MOE_ERR_INVALID_ARG,
                "moe_combine: row size %zu bytes is not a multiple of 16", (size_t)d * esz);
    MOE_REQUIRE(aligned16(y_perm) && aligned16(x) && aligned16(out), MOE_ERR_INVALID_ARG,
                "moe_combine: tensor misaligned");
    return MOE_OK;
}

extern "C" int moe_combine(const void *y_perm, const void *x, const int32_t *inv, const float *expert_prob,
                           int T, int d, int dtype, int residual, void *out, void *stream)
{
    const int rc = combine_check(y_perm, x, inv, expert_prob, T, d, dtype, residual, out);
    if (rc != MOE_OK || T == 0) return rc;
    const size_t esz = dtype == MOE_F32 ? 4 : 2;
    int vec_per_row = (int)((size_t)d * esz / 16);
    hipStream_t st = (hipStream_t)stream;
    const bool big = (size_t)T * vec_per_row * 16 >= CMB_STREAM_BYTES;
    const int lg = combine_lanes(T, vec_per_row);
#define MOE_CMB(B, R)                                                                                              \
    (lg < 0 ? (big ? combine_kernel<B, R, true, CMB_PIECES> : combine_kernel<B, R, false, CMB_PIECES>)             \
            : (big ? combine_kernel<B, R, true, 1> : combine_kernel<B, R, false, 1>))
    auto kern = dtype == MOE_BF16 ? (residual ? MOE_CMB(true, true) : MOE_CMB(true, false))
                                  : (residual ? MOE_CMB(false, true) : MOE_CMB(false, false));
#undef MOE_CMB
    hipLaunchKernelGGL(kern, rows_grid(T, lg < 0 ? 5 : lg), dim3(CMB_THREADS), 0, st, (const cmb_u32x4_t *)y_perm,
                       (const cmb_u32x4_t *)x, inv, expert_prob, T, vec_per_row, lg, (cmb_u32x4_t *)out);
    MOE_CHECK_LAUNCH("moe_combine");
    return MOE_OK;
}

extern "C" int moe_combine_topk(const void *y_perm, const void *x, const int32_t *inv, const float *expert_weight,
                                int T, int k, int d, int dtype, int residual, void *out, void *stream)
{
    MOE_REQUIRE(T >= 0 && d > 0 && k >= 1 && k <= MOE_MAX_TOPK, MOE_ERR_INVALID_ARG,
                "moe_combine_topk: T=%d d=%d k=%d out of range (k <= %d)", T, d, k, MOE_MAX_TOPK);
    MOE_REQUIRE(dtype == MOE_F32 || dtype == MOE_BF16, MOE_ERR_INVALID_ARG, "moe_combine_topk: unknown dtype %d",
                dtype);
    MOE_REQUIRE(residual == 0 || residual == 1, MOE_ERR_INVALID_ARG, "moe_combine_topk: residual must be 0 or 1");
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(y_perm && x && inv && expert_weight && out, MOE_ERR_INVALID_ARG, "moe_combine_topk: null pointer");
    MOE_REQUIRE(out != x && out != y_perm, MOE_ERR_INVALID_ARG, "moe_combine_topk: out aliases an input");
    size_t esz = dtype == MOE_F32 ? 4 : 2;
    MOE_REQUIRE(((size_t)d * esz) % 16 == 0, MOE_ERR_INVALID_ARG,
                "moe_combine_topk: row size %zu bytes is not a multiple of 16", (size_t)d * esz);
    MOE_REQUIRE(aligned16(y_perm) && aligned16(x) && aligned16(out), MOE_ERR_INVALID_ARG,
                "moe_combine_topk: tensor misaligned");
    int vec_per_row = (int)((size_t)d * esz / 16);
    hipStream_t st = (hipStream_t)stream;
    const int lg = combine_topk_lanes(T, vec_per_row);
    auto kern = dtype == MOE_BF16 ? (residual ? combine_topk_kernel<true, true> : combine_topk_kernel<true, false>)
                                  : (residual ? combine_topk_kernel<false, true> : combine_topk_kernel<false, false>);
    hipLaunchKernelGGL(kern, rows_grid(T, lg), dim3(CMB_THREADS), 0, st, (const cmb_u32x4_t *)y_perm,
                       (const cmb_u32x4_t *)x, inv, expert_weight, T, k, vec_per_row, lg, (cmb_u32x4_t *)out);
    MOE_CHECK_LAUNCH("moe_combine_topk");
    return MOE_OK;
}
