// moe_dispatch: capacity-limited, stable dispatch of tokens to expert slots.
//
// Batches of a few thousand entries take the one workgroup of dispatch_small (front.hip) for the tables.  Others:
// three kernels, no global atomics, so the permutation is the stable one whatever the
// hardware scheduling:
//   hist     one workgroup per 1024 tokens: LDS histogram of expert ids -> block_hist[b][e]
//   permute  one workgroup of 1024 threads per 1024 tokens: per expert, total and prefix over the earlier token blocks
//            (the blocks dealt to 1 .. 16 threads per expert, 16 blocks in flight each: one memory round trip up to
//            256 blocks with 64 experts, 64 with 256, 16 with 1024),
//            kept counts, expert offsets (scan over experts), slot offsets (balanced split
//            per expert); then the rank of every token among the tokens of its expert
//            = prefix over earlier blocks + prefix over earlier 64-token chunks of the block
//            (LDS table) + rank inside the chunk (wavefront ballots, one per id bit);
//            writes inv / perm
//            Latency is all it is (one round trip for the loads, one for the stores, a dozen steps in LDS between): with 256 threads, whose
//            histogram sums were four trips and whose ranks four rounds, 65536 ids over 256 experts took 20.8 us with the plan (64 slots) and
//            16.6 without, hist included; now 14.2 and 10.1.
//   gather   whole-chip copy of the kept rows, x_perm[pos] = x[perm[pos]], 16-byte accesses
#include <mutex>

#include "plan_alloc.h"
#include "route.h"

namespace moe {

constexpr int DSP_THREADS = 256;
constexpr int DSP_TOKENS = 1024;  // tokens per workgroup
constexpr int DSP_CHUNKS = DSP_TOKENS / WAVE;

// lanes of the wavefront with this lane's id (0 for an id that does not count)
__device__ __forceinline__ unsigned long long same_id_lanes(int e, bool valid, int nbits)
{
    unsigned long long mask = __ballot(valid);
    for (int b = 0; b < nbits; ++b) {
        const bool bit = (e >> b) & 1;
        const unsigned long long bal = __ballot(bit);
        mask &= bit ? bal : ~bal;
    }
    return valid ? mask : 0ull;
}

// ids that share a wavefront are counted with ballots: a hot expert does not serialise the LDS atomics
__global__ __launch_bounds__(DSP_TOKENS) void dispatch_hist_kernel(const int32_t *__restrict__ idx, int T, int E, int nbits,
                                                                   int32_t *__restrict__ block_hist)
{
    __shared__ int hist[MOE_MAX_EXPERTS];
    const int tid = threadIdx.x, t = blockIdx.x * DSP_TOKENS + tid;
    const int e = t < T ? idx[t] : -1;
    if (tid < E) hist[tid] = 0;
    __syncthreads();
    const unsigned long long mask = same_id_lanes(e, e >= 0 && e < E, nbits);
    if (mask && (mask & ((1ull << (tid & 63)) - 1ull)) == 0) atomicAdd(&hist[e], __popcll(mask));
    __syncthreads();
    if (tid < E) block_hist[(size_t)blockIdx.x * E + tid] = hist[tid];
}

// Exclusive scans of two values per thread over the workgroup of 1024; sums: LDS scratch of 32 ints.
__device__ __forceinline__ void block_scan2_1024(int v0, int v1, int &ex0, int &ex1, int &tot0, int &tot1, int *sums)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i0 = wave_scan_incl(v0), i1 = wave_scan_incl(v1);
    if (lane == 63) {
        sums[w] = i0;
        sums[16 + w] = i1;
    }
    __syncthreads();
    int b0 = 0, b1 = 0;
    tot0 = tot1 = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int a = sums[i], b = sums[16 + i];
        b0 += i < w ? a : 0;
        b1 += i < w ? b : 0;
        tot0 += a;
        tot1 += b;
    }
    ex0 = b0 + i0 - v0;
    ex1 = b1 + i1 - v1;
}

// One workgroup per 1024 tokens.  Every workgroup first rebuilds, from the per-block
// histograms, the per-expert totals, its own prefix over earlier blocks, the kept counts and
// the expert offsets (a few KB of reads; cheaper than a separate single-workgroup launch in
// the dependency chain); workgroup 0 also writes those tables and the slot offsets out.
//
// PPL > 0: the replica plan is made here as well (PPL = experts per lane of the allocating wavefront), by
// every workgroup for itself from the same counts -- the plan's own ids' histograms in plan_partial, or, when
// that is NULL, the routed ids' totals just rebuilt (a plan made from the routed ids themselves) -- so the
// plan kernels and their place in the dependency chain go away; workgroup 0 writes the plan's tables.
struct PlanArgs {
    const int32_t *plan_partial;
    int n_partial, n_plan_ids, R, policy;
    int32_t *plan_counts, *replicas, *slot_base, *slot_expert, *n_slots;
};

template <int PPL>
__global__ __launch_bounds__(DSP_TOKENS) void dispatch_permute_kernel(
    const int32_t *__restrict__ idx, const int32_t *__restrict__ replicas, int T, int E, int nbits, int C, int nb,
    int max_slots, const int32_t *__restrict__ block_hist, int32_t *__restrict__ counts, int32_t *__restrict__ kept,
    int32_t *__restrict__ expert_offset, int32_t *__restrict__ slot_offset, int32_t *__restrict__ perm,
    int32_t *__restrict__ inv, int n_tokens, int32_t *__restrict__ row_token, PlanArgs pa)
{
    __shared__ unsigned short chunk_cnt[DSP_CHUNKS][MOE_MAX_EXPERTS];
    __shared__ int before_e[MOE_MAX_EXPERTS];   // tokens of e in earlier blocks
    __shared__ int tot_e[MOE_MAX_EXPERTS];      // and in all
    __shared__ int eoff_e[MOE_MAX_EXPERTS];     // first permuted row of e
    __shared__ int cap_e[MOE_MAX_EXPERTS];      // kept count of e
    __shared__ int sums[32];
    __shared__ int plan_hist[PPL > 0 ? MOE_MAX_EXPERTS : 1];
    __shared__ int rep[PPL > 0 ? MOE_MAX_EXPERTS : 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;

    // ---- Everything this workgroup reads is asked for up front: its tokens' ids, and the block histograms, (expert, part of the blocks)
    // per thread.
    const int t = blockIdx.x * DSP_TOKENS + tid;
    int id = t < T ? idx[t] : -1;
    const int given = PPL == 0 && replicas && tid < E ? replicas[tid] : 1;
    const int n_parts = E <= DSP_TOKENS / 16 ? 16 : E <= DSP_TOKENS / 8 ? 8 : E <= DSP_TOKENS / 4 ? 4 : E <= DSP_TOKENS / 2 ? 2 : 1;
    const int span = DSP_TOKENS / n_parts, e_own = tid % span, part = tid / span;     // powers of two
    int tot = 0, bef = 0;
    if (e_own < E) {
#pragma unroll 16
        for (int b = part; b < nb; b += n_parts) {
            const int v = block_hist[(size_t)b * E + e_own];
            bef += b < (int)blockIdx.x ? v : 0;
            tot += v;
        }
    }
    int planned = 0;
    if (PPL > 0 && pa.plan_partial && e_own < E)
        for (int b = part; b < pa.n_partial; b += n_parts) planned += pa.plan_partial[(size_t)b * E + e_own];
    for (int i = tid; i < DSP_CHUNKS * E; i += DSP_TOKENS) chunk_cnt[i / E][i % E] = 0;
    before_e[tid] = 0;
    tot_e[tid] = 0;
    if (PPL > 0) plan_hist[tid] = 0;
    __syncthreads();
    if (e_own < E) {
        if (tot) atomicAdd(&tot_e[e_own], tot);
        if (bef) atomicAdd(&before_e[e_own], bef);
        if (PPL > 0) {
            const int h = pa.plan_partial ? planned : tot;
            if (h) atomicAdd(&plan_hist[e_own], h);
        }
    }
    // ---- rank of every token inside its wavefront's 64
    const bool valid = id >= 0 && id < E;
    const unsigned long long mask = same_id_lanes(id, valid, nbits);
    const int rank = __popcll(mask & ((1ull << lane) - 1ull));
    if (valid && rank == 0) chunk_cnt[w][id] = (unsigned short)__popcll(mask);
    __syncthreads();

    // ---- wavefront 0: the plan; the others: per expert, prefix of the chunk counts
    if (PPL > 0 && tid < WAVE) {
        plan_allocate_wave<(PPL > 0 ? PPL : 1)>(plan_hist, rep, pa.n_plan_ids, E, pa.R, C, pa.policy, pa.replicas, pa.plan_counts,
                                                blockIdx.x == 0);
    } else {
        constexpr int FIRST = PPL > 0 ? WAVE : 0;
        for (int e = tid - FIRST; e < E; e += DSP_TOKENS - FIRST) {
            int v[DSP_CHUNKS];
#pragma unroll
            for (int c = 0; c < DSP_CHUNKS; ++c) v[c] = chunk_cnt[c][e];
            int run = 0;
#pragma unroll
            for (int c = 0; c < DSP_CHUNKS; ++c) {
                chunk_cnt[c][e] = (unsigned short)run;
                run += v[c];
            }
        }
    }
    if (PPL > 0) __syncthreads();
    // ---- thread e owns expert e
    const int r_e = tid < E ? (PPL > 0 ? rep[tid] : given < 1 ? 1 : given) : 0;
    const int n_e = tid < E ? tot_e[tid] : 0;
    const long long cap = (long long)r_e * C;
    const int k_e = (long long)n_e < cap ? n_e : (int)cap;
    int off_e, sb_e, K, P;
    // more replicas than the slot tables hold count as one more: a caller's may be any number, and their sum has to fit
    block_scan2_1024(k_e, r_e > max_slots ? max_slots + 1 : r_e, off_e, sb_e, K, P, sums);
    if (tid < E) {
        eoff_e[tid] = off_e;
        cap_e[tid] = k_e;
    }
    __syncthreads();
    if (T > 0) {
        int dest = -1;
        if (valid) {
            const int j = before_e[id] + chunk_cnt[w][id] + rank;
            if (j < cap_e[id]) dest = eoff_e[id] + j;
        }
        if (t < T) {
            inv[t] = dest;
            if (dest >= 0) perm[dest] = t;
            if (t >= K) perm[t] = -1;
            if (row_token) {            // top-k: entry t is assignment (t / n_tokens, t % n_tokens)
                if (dest >= 0) row_token[dest] = t % n_tokens;
                if (t >= K) row_token[t] = -1;
            }
        }
    }
    if (blockIdx.x != 0) return;
    if (tid < E) {
        counts[tid] = n_e;
        kept[tid] = k_e;
        expert_offset[tid] = off_e;
        if (PPL > 0 && pa.slot_base) pa.slot_base[tid] = sb_e;
    }
    // slot tables: an expert's slots are written by its whole wavefront, 64 at a time, those that the tables hold
    const int q = r_e > 0 ? k_e / r_e : 0, rem = r_e > 0 ? k_e % r_e : 0;
    auto write_slot = [&](int e, int p, int k, int first, int quot, int rest) {
        if (slot_offset) slot_offset[p] = first + k * quot + (k < rest ? k : rest);
        if (PPL > 0 && pa.slot_expert) pa.slot_expert[p] = e;
    };
    if (r_e > 0 && sb_e <= max_slots) write_slot(tid, sb_e, 0, off_e, q, rem);
    for (unsigned long long more = __ballot(r_e > 1); more; more &= more - 1) {
        const int l = __builtin_ctzll(more);                     // uniform
        const int r = __builtin_amdgcn_readlane(r_e, l), p0 = __builtin_amdgcn_readlane(sb_e, l);
        const int first = __builtin_amdgcn_readlane(off_e, l), quot = __builtin_amdgcn_readlane(q, l);
        const int rest = __builtin_amdgcn_readlane(rem, l);
        const int last = p0 > max_slots ? 0 : r - 1 < max_slots - p0 ? r - 1 : max_slots - p0;
        for (unsigned k = 1 + lane; k <= (unsigned)last; k += WAVE) write_slot(w * WAVE + l, p0 + (int)k, (int)k, first, quot, rest);
    }
    if (tid == 0) {
        expert_offset[E] = K;
        if (PPL > 0 && pa.slot_base) pa.slot_base[E] = P;
        if (PPL > 0 && pa.n_slots) pa.n_slots[0] = P;
    }
    if (slot_offset)
        for (int p = P + tid; p <= max_slots; p += DSP_TOKENS) slot_offset[p] = K;
    if (PPL > 0 && pa.slot_expert)
        for (int p = P + tid; p < E + pa.R; p += DSP_TOKENS) pa.slot_expert[p] = -1;
}

// x_perm[pos] = x[perm[pos]] for pos < K (K is not read: the permutation ends in -1 entries).  32 lanes per row, 8 rows per workgroup, 16-byte
// pieces: the scattered row reads and the contiguous writes are both whole lines, the row
// index is read once per row, and a lane's three loads of a trip are independent.
// STREAM: an output far beyond what the L2s hold is written past them (combine.hip: where the line lies, and what it costs a reader
// that follows at once).  Measured, 65536 x 768 bf16: 47 -> 37 us (30 us alone, 6.7 TB/s) on top of
// the tables; 16384 tokens 16 -> 8.6 us (a trip of four pieces that rows of 96 never fill took the leftover path before).
constexpr int GATHER_ROWS = DSP_THREADS / 32;
constexpr size_t GATHER_STREAM_BYTES = (size_t)64 << 20;
typedef unsigned dsp_u32x4_t __attribute__((ext_vector_type(4)));

template <bool STREAM>
__global__ __launch_bounds__(DSP_THREADS) void dispatch_gather_kernel(const dsp_u32x4_t *__restrict__ x,
                                                                      const int32_t *__restrict__ perm, int T,
                                                                      int n_tokens, int vec_per_row,
                                                                      dsp_u32x4_t *__restrict__ x_perm)
{
    const int pos = blockIdx.x * GATHER_ROWS + (threadIdx.x >> 5);
    const int l = threadIdx.x & 31;
    if (pos >= T) return;
    int row = perm[pos];
    if (row < 0) return;                      // past the kept rows (perm holds -1 there): nothing to copy
    if (row >= n_tokens) row %= n_tokens;     // top-k: assignment -> its token
    const dsp_u32x4_t *src = x + (size_t)row * vec_per_row;
    dsp_u32x4_t *dst = x_perm + (size_t)pos * vec_per_row;
    for (int c = l; c < vec_per_row; c += 96) {
        dsp_u32x4_t v[3];
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (c + u * 32 < vec_per_row) v[u] = src[c + u * 32];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            if (c + u * 32 >= vec_per_row) continue;
            if (STREAM) __builtin_nontemporal_store(v[u], dst + c + u * 32);
            else dst[c + u * 32] = v[u];
        }
    }
}

size_t dispatch_block_hist_bytes(int T, int E)
{
    size_t nb = (size_t)ceil_div(T, DSP_TOKENS);
    return align_up((nb > 0 ? nb : 1) * (size_t)E * sizeof(int32_t), 256);
}

int dispatch_planned_launch(const int32_t *expert_idx, int T, int n_tokens, int E, int slot_capacity, int budget,
                            int policy, const int32_t *plan_partial, int n_partial, int n_plan_ids,
                            int32_t *block_hist, int32_t *plan_counts, int32_t *replicas, int32_t *slot_base,
                            int32_t *slot_expert, int32_t *n_slots, int32_t *counts, int32_t *kept,
                            int32_t *expert_offset, int32_t *slot_offset, int32_t *perm, int32_t *inv,
                            int32_t *row_token, hipStream_t st, const char *who)
{
    const int nb = ceil_div(T, DSP_TOKENS);
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    if (nb > 0) {
        hipLaunchKernelGGL(dispatch_hist_kernel, dim3(nb), dim3(DSP_TOKENS), 0, st, expert_idx, T, E, nbits, block_hist);
        MOE_CHECK_LAUNCH(who);
    }
    PlanArgs pa{plan_partial, n_partial, n_plan_ids, budget, policy, plan_counts, replicas, slot_base, slot_expert,
                n_slots};
    // With 16 experts per lane the plan keeps 49 of its registers in scratch (1024 threads leave 128 each; with 256 it had 206), and is ahead
    // all the same: 30000 ids, 512 experts, 64 slots 43.9 us with 256 threads and slots one by one, 26.4 now.
    auto kern = E <= 128 ? dispatch_permute_kernel<2> : E <= 256 ? dispatch_permute_kernel<4> : dispatch_permute_kernel<16>;
    hipLaunchKernelGGL(kern, dim3(nb > 0 ? nb : 1), dim3(DSP_TOKENS), 0, st, expert_idx, (const int32_t *)nullptr, T, E,
                       nbits, slot_capacity, nb, E + budget, block_hist, counts, kept, expert_offset, slot_offset, perm,
                       inv, n_tokens > 0 ? n_tokens : 1, row_token, pa);
    MOE_CHECK_LAUNCH(who);
    return MOE_OK;
}

// ------------------------------------------------------------------ allocation-free variant
// The per-block histograms of moe_dispatch_static live in this file-scope device array instead of a
// caller's workspace.  Every GPU the library runs on holds its own copy at its own address until the
// process ends.  In host code the array's name is only a stand-in for the symbol: its device address is
// asked of the runtime once per device and that pointer is what the kernels get.
constexpr size_t DSP_STATIC_BYTES = (size_t)1 << 20;   // 262144 table entries: e.g. 256 blocks x 1024 experts
static __device__ __align__(256) int32_t scratch[DSP_STATIC_BYTES / sizeof(int32_t)];

constexpr int DSP_MAX_DEVICES = 64;
static std::mutex g_scratch_mutex;
static int32_t *g_scratch_ptr[DSP_MAX_DEVICES];        // device address of `scratch` per device ordinal

static int32_t *static_scratch_of_current_device(const char *who)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= DSP_MAX_DEVICES) {
        set_error("%s: cannot tell the current device (ordinal %d, at most %d devices)", who, dev, DSP_MAX_DEVICES);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            set_error("%s: hipGetSymbolAddress(scratch) failed on device %d: %s", who, dev, hipGetErrorString(e));
            return nullptr;
        }
        g_scratch_ptr[dev] = (int32_t *)p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace moe

using namespace moe;

extern "C" size_t moe_dispatch_workspace_bytes(int T, int E)
{
    if (T < 0 || E <= 0) return 0;
    size_t nb = (size_t)ceil_div(T, DSP_TOKENS);
    return align_up((nb > 0 ? nb : 1) * (size_t)E * sizeof(int32_t), 256);
}

// T entries (tokens, or k*n_tokens assignments of a top-k layer) over the rows of n_tokens tokens
static int dispatch_checked(const char *who, const void *x, const int32_t *expert_idx, const int32_t *replicas, int T,
                            int n_tokens, int d, int E, int slot_capacity, int max_slots, int dtype, int32_t *counts,
                            int32_t *kept, int32_t *expert_offset, int32_t *slot_offset, int32_t *perm, int32_t *inv,
                            int32_t *row_token, void *x_perm, void *ws, size_t ws_bytes, void *stream,
                            bool static_scratch = false)
{
    MOE_REQUIRE(T >= 0 && d > 0 && E > 0 && slot_capacity >= 1 && max_slots >= 0, MOE_ERR_INVALID_ARG,
                "%s: T=%d d=%d E=%d slot_capacity=%d max_slots=%d out of range", who, T, d, E, slot_capacity,
                max_slots);
    MOE_REQUIRE(dtype == MOE_F32 || dtype == MOE_BF16, MOE_ERR_INVALID_ARG, "%s: unknown dtype %d", who, dtype);
    MOE_REQUIRE(E <= MOE_MAX_EXPERTS, MOE_ERR_UNSUPPORTED, "%s: E=%d exceeds %d", who, E, MOE_MAX_EXPERTS);
    MOE_REQUIRE(counts && kept && expert_offset && (T == 0 || (expert_idx && perm && inv)), MOE_ERR_INVALID_ARG,
                "%s: null output or id pointer", who);
    MOE_REQUIRE((x == nullptr) == (x_perm == nullptr), MOE_ERR_INVALID_ARG,
                "%s: x and x_perm must both be given or both be NULL", who);
    MOE_REQUIRE(!slot_offset || max_slots >= E, MOE_ERR_INVALID_ARG, "%s: max_slots=%d smaller than E=%d", who,
                max_slots, E);
    size_t esz = dtype == MOE_F32 ? 4 : 2;
    MOE_REQUIRE(((size_t)d * esz) % 16 == 0, MOE_ERR_INVALID_ARG, "%s: row size %zu bytes is not a multiple of 16",
                who, (size_t)d * esz);
    MOE_REQUIRE(aligned16(x) && aligned16(x_perm), MOE_ERR_INVALID_ARG, "%s: x / x_perm misaligned", who);
    if (static_scratch) {
        MOE_REQUIRE(moe_dispatch_workspace_bytes(T, E) <= DSP_STATIC_BYTES, MOE_ERR_UNSUPPORTED,
                    "%s: ceil(T/1024)*E = %zu table entries exceed the %zu of the static scratch array "
                    "(use moe_dispatch with a workspace)",
                    who, moe_dispatch_workspace_bytes(T, E) / sizeof(int32_t), DSP_STATIC_BYTES / sizeof(int32_t));
        ws = static_scratch_of_current_device(who);
        if (!ws) return MOE_ERR_HIP;
    } else {
        MOE_REQUIRE(ws && ws_bytes >= moe_dispatch_workspace_bytes(T, E), MOE_ERR_WORKSPACE,
                    "%s: workspace of %zu bytes needed, %zu given", who, moe_dispatch_workspace_bytes(T, E), ws_bytes);
    }
    hipStream_t st = (hipStream_t)stream;
    int nb = ceil_div(T, DSP_TOKENS);
    int32_t *block_hist = (int32_t *)ws;
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    if (dispatch_small(T, E)) {
        const int rc = dispatch_small_launch(expert_idx, replicas, T, n_tokens, E, slot_capacity, max_slots, counts, kept, expert_offset,
                                             slot_offset, perm, inv, row_token, st, who);
        if (rc != MOE_OK) return rc;
    } else {
        if (nb > 0) {
            hipLaunchKernelGGL(dispatch_hist_kernel, dim3(nb), dim3(DSP_TOKENS), 0, st, expert_idx, T, E, nbits, block_hist);
            MOE_CHECK_LAUNCH(who);
        }
        hipLaunchKernelGGL(dispatch_permute_kernel<0>, dim3(nb > 0 ? nb : 1), dim3(DSP_TOKENS), 0, st, expert_idx,
                           replicas, T, E, nbits, slot_capacity, nb, max_slots, block_hist, counts, kept,
                           expert_offset, slot_offset, perm, inv, n_tokens > 0 ? n_tokens : 1, row_token, PlanArgs{});
        MOE_CHECK_LAUNCH(who);
    }
    if (x && nb > 0) {
        int vec_per_row = (int)((size_t)d * esz / 16);
        int grid = ceil_div(T, GATHER_ROWS);
        auto gather = (size_t)T * vec_per_row * 16 >= GATHER_STREAM_BYTES ? dispatch_gather_kernel<true>
                                                                          : dispatch_gather_kernel<false>;
        hipLaunchKernelGGL(gather, dim3(grid), dim3(DSP_THREADS), 0, st, (const dsp_u32x4_t *)x, perm, T, n_tokens,
                           vec_per_row, (dsp_u32x4_t *)x_perm);
        MOE_CHECK_LAUNCH(who);
    }
    return MOE_OK;
}

extern "C" int moe_dispatch(const void *x, const int32_t *expert_idx, const int32_t *replicas, int T, int d,
                            int E, int slot_capacity, int max_slots, int dtype, int32_t *counts,
                            int32_t *kept, int32_t *expert_offset, int32_t *slot_offset, int32_t *perm,
                            int32_t *inv, void *x_perm, void *ws, size_t ws_bytes, void *stream)
{
    return dispatch_checked("moe_dispatch", x, expert_idx, replicas, T, T, d, E, slot_capacity, max_slots, dtype,
                            counts, kept, expert_offset, slot_offset, perm, inv, nullptr, x_perm, ws, ws_bytes, stream);
}

extern "C" int moe_dispatch_topk(const void *x, const int32_t *expert_idx, const int32_t *replicas, int T, int k,
                                 int d, int E, int slot_capacity, int max_slots, int dtype, int32_t *counts,
                                 int32_t *kept, int32_t *expert_offset, int32_t *slot_offset, int32_t *perm,
                                 int32_t *inv, int32_t *row_token, void *x_perm, void *ws, size_t ws_bytes,
                                 void *stream)
{
    MOE_REQUIRE(T >= 0 && k >= 1 && k <= MOE_MAX_TOPK && (long long)T * k <= 0x7fffffffLL, MOE_ERR_INVALID_ARG,
                "moe_dispatch_topk: T=%d k=%d out of range (k <= %d, T*k < 2^31)", T, k, MOE_MAX_TOPK);
    MOE_REQUIRE(T == 0 || row_token, MOE_ERR_INVALID_ARG, "moe_dispatch_topk: null row_token");
    return dispatch_checked("moe_dispatch_topk", x, expert_idx, replicas, T * k, T, d, E, slot_capacity, max_slots,
                            dtype, counts, kept, expert_offset, slot_offset, perm, inv, row_token, x_perm, ws, ws_bytes,
                            stream);
}

extern "C" int moe_dispatch_static(const void *x, const int32_t *expert_idx, const int32_t *replicas, int T, int d,
                                   int E, int slot_capacity, int max_slots, int dtype, int32_t *counts,
                                   int32_t *kept, int32_t *expert_offset, int32_t *slot_offset, int32_t *perm,
                                   int32_t *inv, void *x_perm, void *stream)
{
    return dispatch_checked("moe_dispatch_static", x, expert_idx, replicas, T, T, d, E, slot_capacity, max_slots,
                            dtype, counts, kept, expert_offset, slot_offset, perm, inv, nullptr, x_perm, nullptr, 0,
                            stream, true);
}
