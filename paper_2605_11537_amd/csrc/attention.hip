// Sparsemax self-attention over the states of the last SRU layer (the predictor's "sparse
// attention": Methodology; SRU subsection, last paragraph).  Per sequence of L positions and
// n features:
//     s[t, j] = <h_t, h_j> / sqrt(n),   a[t, :] = sparsemax(s[t, :]),   z_t = h_t + sum_j a[t, j] h_j
// with sparsemax(s) = max(s - tau, 0), tau such that the entries sum to one (the Euclidean
// projection onto the simplex).  z is stored in bf16 and goes to the predictor's head.
//
// One workgroup = 32 consecutive positions of one sequence.
//   1. scores on the matrix cores: the last layer hands its states over as matrix-core fragments (32 positions x 16
//      features, 1 KB each), which are queries and keys as the instruction wants them; the sequence's states stay in L2 for
//      its 16 workgroups; the 32 x L fp32 score tile is kept in LDS.  (Sequences of fewer than 8 positions come row-major.)
//   2. sparsemax, one wavefront per 4 rows, each lane holding L/64 scores of each: tau by Michelot's
//      fixed point (tau = (sum of the entries above tau - 1) / their count, until the set is stable),
//      which ends at exactly the support the sorting definition gives.  The four rows go through the loop together: a row
//      is a chain of reductions across the wavefront, and one after the other they were the longest part of the kernel.
//   3. the context sum_j a[t, j] h_j on the matrix cores: the contraction runs over positions, so the
//      state operand must have 8 consecutive positions of one feature per lane -- the last layer also writes, per sequence,
//      the packed image of its states as a (positions x features) matrix (the
//      layout moe_pack_weights gives weights: a wavefront's fragment load is 1 KB of consecutive memory).  Its first
//      512 positions are requested before step 2.
//      The weights go back into the score tile and are read from there
//      as the other operand, rounded to bf16 (relative error 2^-9 per weight, the size of the bf16
//      rounding of z itself).  On the vector units the same sum is 16384 multiply-adds per lane and took
//      three times as long as everything else in the kernel.
// Measured, 8 x 512, 256 features: 12.3 us at best, 13 in the predictor, against 23 us and 4 us for the image in a kernel of its own.
#include "gemm_bf16.h"
#include "route.h"

namespace moe {

constexpr int ATT_QT = 32;           // query rows per workgroup
constexpr int ATT_MAX_L = 1024;      // positions per sequence the LDS score tile holds
constexpr int ATT_WAVES = 8;         // wavefronts per workgroup (two per SIMD)
constexpr int ATT_THREADS = ATT_WAVES * 64;

// Wavefront-wide reductions on the data-parallel-primitive path (a cross-lane operand of an ordinary
// vector instruction) instead of LDS-routed shuffles: sparsemax does a dozen of them per row, one
// after the other.  Four steps fold a row of 16 lanes (quad swaps, then rotations by 4 and 8); the
// four row results are read as scalars and added.  Every lane gets the result.
template <class Op>
__device__ __forceinline__ float wave_reduce_f(float v, Op op)
{
    auto dpp = [](float x, int ctrl) {
        switch (ctrl) {
        case 0: return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0xB1, 0xf, 0xf, false));
        case 1: return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x4E, 0xf, 0xf, false));
        case 2: return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x124, 0xf, 0xf, false));
        default: return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x128, 0xf, 0xf, false));
        }
    };
    v = op(v, dpp(v, 0));    // lane ^ 1
    v = op(v, dpp(v, 1));    // lane ^ 2
    v = op(v, dpp(v, 2));    // the quad 4 lanes away in the row of 16
    v = op(v, dpp(v, 3));    // the half row 8 lanes away
    const int b = __builtin_bit_cast(int, v);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 0));
    const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 32));
    const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(b, 48));
    return op(op(r0, r1), op(r2, r3));
}
__device__ __forceinline__ float wave_sum_f(float v) { return wave_reduce_f(v, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float wave_max_f(float v) { return wave_reduce_f(v, [](float a, float b) { return fmaxf(a, b); }); }

typedef unsigned att_u32x4_t __attribute__((ext_vector_type(4)));

// NKS = features / 16.  PER: scores per lane and row, L <= 64 * PER.  FRAG: h is the fragment image of the states, else row-major.
template <int NKS, int PER, bool FRAG>
__global__ __launch_bounds__(ATT_THREADS, 1) void sru_attention_kernel(const bf16_t *__restrict__ h,
                                                                        const bf16_t *__restrict__ hp, int n_units, int L,
                                                                        int Lp, bf16_t *__restrict__ z)
{
    constexpr int n = NKS * 16, LDQ = n + 8, LDS_S = 64 * PER + 4;
    __shared__ __attribute__((aligned(16))) float s_lds[ATT_QT * LDS_S];
    __shared__ __attribute__((aligned(16))) bf16_t q_lds[ATT_QT * LDQ];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // All query blocks of a sequence read the same keys and packed states: 8 contiguous ranges of the (sequence, query block) pairs, one per
    // XCD, so that an XCD's L2 holds the states of about 1/8 of the sequences instead of cycling through all of them.
    const int n_kb = (L + 31) / 32;              // blocks of 32 positions: query blocks and key blocks
    const int unit = xcd_remap(blockIdx.x, n_units);
    if (unit < 0) return;
    const int seq = unit / n_kb, qblk = unit - seq * n_kb;
    const int q0 = qblk * ATT_QT;
    const bf16_t *hs = h + (size_t)seq * L * n;
    const att_u32x4_t *frag = reinterpret_cast<const att_u32x4_t *>(h) + (size_t)seq * n_kb * NKS * 64;
    // Two key blocks of this wavefront at a time (w and w + 8, then w + 16 and w + 24), all their fragments requested at once;
    // a block past the end repeats the last.  Row-major: an operand row is 8 consecutive features per lane.
    att_u32x4_t kf[2][NKS];
    auto load_keys = [&](int kb0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            int kb = kb0 + u * ATT_WAVES;
            kb = kb < n_kb ? kb : n_kb - 1;
            const int key = kb * 32 + (lane & 31) < L ? kb * 32 + (lane & 31) : L - 1;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                kf[u][ks] = FRAG ? frag[((size_t)kb * NKS + ks) * 64 + lane]
                                 : *reinterpret_cast<const att_u32x4_t *>(hs + (size_t)key * n + ks * 16 + (lane >> 5) * 8);
        }
    };
    // query rows (positions past the sequence end: whatever the image holds there, or its last row; they are never stored)
    constexpr int QP = ATT_QT * (n / 8) / ATT_THREADS;       // 16-byte pieces per thread
#pragma unroll
    for (int i = 0; i < QP; ++i) {
        const int p = tid + i * ATT_THREADS, r = p & 31, g = p >> 5;
        const int t = q0 + r < L ? q0 + r : L - 1;
        *reinterpret_cast<att_u32x4_t *>(q_lds + r * LDQ + g * 8) =
            FRAG ? frag[((size_t)qblk * NKS + (g >> 1)) * 64 + (g & 1) * 32 + r]
                 : *reinterpret_cast<const att_u32x4_t *>(hs + (size_t)t * n + g * 8);
    }
    load_keys(w);
    __syncthreads();
    // 1. scores
    const float scale = rsqrtf((float)n);
    for (int kb0 = w; kb0 < n_kb; kb0 += 2 * ATT_WAVES) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int kb = kb0 + u * ATT_WAVES;
            if (kb >= n_kb) break;               // uniform
            f32x16_t acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.f;
            const bf16_t *qrow = q_lds + (lane & 31) * LDQ + (lane >> 5) * 8;
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const att_u32x4_t *>(qrow + ks * 16)),
                    __builtin_bit_cast(bf16x8_t, kf[u][ks]), acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 16; ++v) s_lds[acc_row(v, lane) * LDS_S + kb * 32 + (lane & 31)] = acc[v] * scale;
        }
        if (kb0 + 2 * ATT_WAVES < n_kb) load_keys(kb0 + 2 * ATT_WAVES);
    }
    // fragments of the packed states for step 3 (feature block w), positions 16 SB (b) + 16 u; past the end the last again
    constexpr int SB = PER * 4 < 32 ? PER * 4 : 32;          // fragments in flight
    const bool have = w * 32 < n;                            // uniform
    const att_u32x4_t *st = reinterpret_cast<const att_u32x4_t *>(hp) +
                            ((size_t)seq * (n / 32) + (have ? w : 0)) * (Lp / 8) * 32 + lane;
    att_u32x4_t sf[SB];
    auto load_state = [&](int step, int u) {
        const int last = Lp / 16 - 1;
        sf[u] = st[(size_t)(step < last ? step : last) * 64];
    };
#pragma unroll
    for (int u = 0; u < SB; ++u) load_state(u, u);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // 2. sparsemax: this wavefront's four rows together
    {
        constexpr int RW = ATT_QT / ATT_WAVES;
        float zr[RW][PER], tau[RW], cnt[RW], mx[RW], sum[RW];
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            const float *row = s_lds + (w * RW + rr) * LDS_S;
            mx[rr] = -INFINITY;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                const int j = i * 64 + lane;
                zr[rr][i] = j < L ? row[j] : -INFINITY;
                mx[rr] = fmaxf(mx[rr], zr[rr][i]);
            }
        }
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) mx[rr] = wave_max_f(mx[rr]);
        // shift by the row maximum (sparsemax is shift invariant): the sums below stay small
        // counts are kept as floats (exact up to 2^24) so that one reduction serves sums and counts alike
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            sum[rr] = cnt[rr] = 0.f;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
                zr[rr][i] -= mx[rr];                // -inf stays -inf
                if (zr[rr][i] > -INFINITY) {
                    sum[rr] += zr[rr][i];
                    cnt[rr] += 1.f;
                }
            }
        }
        bool open[RW];
        bool any = false;
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            sum[rr] = wave_sum_f(sum[rr]);
            cnt[rr] = wave_sum_f(cnt[rr]);
            tau[rr] = (sum[rr] - 1.f) / cnt[rr];
            open[rr] = q0 + w * RW + rr < L;        // uniform: rows past the sequence are not looked at
            any = any || open[rr];
        }
        while (any) {
            float s2[RW], c2[RW];
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) {
                s2[rr] = c2[rr] = 0.f;
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    if (zr[rr][i] > tau[rr]) {
                        s2[rr] += zr[rr][i];
                        c2[rr] += 1.f;
                    }
            }
            any = false;
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) {
                s2[rr] = wave_sum_f(s2[rr]);
                c2[rr] = wave_sum_f(c2[rr]);
                // the set above tau did not shrink: tau is final.  c2 is never 0: the maximum (0 after the shift) stays above tau < 0
                open[rr] = open[rr] && c2[rr] < cnt[rr];
                if (open[rr]) {
                    cnt[rr] = c2[rr];
                    tau[rr] = (s2[rr] - 1.f) / c2[rr];
                }
                any = any || open[rr];
            }
        }
        // the weights go back into the rows of the score tile (positions past the sequence, and rows past it, get 0)
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            float *row = s_lds + (w * RW + rr) * LDS_S;
            const bool in = q0 + w * RW + rr < L;
#pragma unroll
            for (int i = 0; i < PER; ++i) row[i * 64 + lane] = in && zr[rr][i] > tau[rr] ? zr[rr][i] - tau[rr] : 0.f;
        }
    }
    __syncthreads();   // every row's weights are in the score tile
    // 3. context on the matrix cores: wavefront w owns feature block w (32 features) of all
    // 32 rows; per step of 16 positions one weight fragment (from the score tile, rounded to bf16) and one
    // fragment of the packed states.
    if (have) {
        f32x16_t acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const float *arow = s_lds + (lane & 31) * LDS_S + (lane >> 5) * 8;
        auto context_step = [&](int step, int u) {
            const float4 a_lo = *reinterpret_cast<const float4 *>(arow + step * 16);
            const float4 a_hi = *reinterpret_cast<const float4 *>(arow + step * 16 + 4);
            uint4 af;
            af.x = pack_bf16x2(a_lo.x, a_lo.y);
            af.y = pack_bf16x2(a_lo.z, a_lo.w);
            af.z = pack_bf16x2(a_hi.x, a_hi.y);
            af.w = pack_bf16x2(a_hi.z, a_hi.w);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, af),
                                                          __builtin_bit_cast(bf16x8_t, sf[u]), acc, 0, 0, 0);
        };
        const int steps = Lp / 16;
#pragma unroll
        for (int u = 0; u < SB; ++u)
            if (u < steps) context_step(u, u);               // uniform
        if constexpr (PER * 4 > SB) {                        // the second half of the longest sequences
            if (steps > SB) {
#pragma unroll
                for (int u = 0; u < SB; ++u) load_state(SB + u, u);
#pragma unroll
                for (int u = 0; u < SB; ++u)
                    if (SB + u < steps) context_step(SB + u, u);
            }
        }
        const int f = w * 32 + (lane & 31);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = acc_row(v, lane);
            if (q0 + r < L)
                z[((size_t)seq * L + q0 + r) * n + f] = f32_to_bf16(bf16_to_f32(q_lds[r * LDQ + f]) + acc[v]);
        }
    }
}

// h [B*L, n] -> per sequence the packed image of the (Lp x n) matrix of its states (positions past L are
// zero): 16-byte piece ((f / 32) * (Lp / 8) + t / 8) * 32 + f % 32 holds h[8 (t / 8) .. + 7][f]
__global__ __launch_bounds__(256) void sru_pack_states_kernel(const bf16_t *__restrict__ h, int L, int Lp, int n,
                                                              uint4 *__restrict__ hp)
{
    const int per_seq = (n / 32) * (Lp / 8) * 32;
    const int p = blockIdx.x * 256 + threadIdx.x, seq = blockIdx.y;
    if (p >= per_seq) return;
    const int c = p & 31, kg = (p >> 5) % (Lp / 8), strip = (p >> 5) / (Lp / 8);
    const bf16_t *src = h + ((size_t)seq * L + kg * 8) * n + strip * 32 + c;
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = kg * 8 + 2 * i;
        const uint32_t lo = t < L ? src[(size_t)(2 * i) * n] : 0, hi = t + 1 < L ? src[(size_t)(2 * i + 1) * n] : 0;
        v[i] = lo | (hi << 16);
    }
    hp[(size_t)seq * per_seq + p] = make_uint4(v[0], v[1], v[2], v[3]);
}

size_t sru_attention_ws_bytes(int B, int L, int n) { return align_up((size_t)(B > 0 ? B : 1) * n * align_up((size_t)L, 16) * 2, 256); }

bool sru_attention_takes_fragments(int L) { return L >= 8; }

int sru_attention_launch(const void *h, bool fragments, int B, int L, int n, void *z, void *ht_ws, hipStream_t st,
                         const char *who)
{
    MOE_REQUIRE(L <= ATT_MAX_L && (n == 128 || n == 256), MOE_ERR_UNSUPPORTED,
                "%s: sparsemax attention is built for L <= %d and n_hidden = 128 or 256; got L=%d n_hidden=%d", who,
                ATT_MAX_L, L, n);
    if (B == 0) return MOE_OK;
    const int Lp = (int)align_up((size_t)L, 16);
    if (!fragments) {
        hipLaunchKernelGGL(sru_pack_states_kernel, dim3(ceil_div((n / 32) * (Lp / 8) * 32, 256), B), dim3(256), 0, st,
                           (const bf16_t *)h, L, Lp, n, (uint4 *)ht_ws);
        MOE_CHECK_LAUNCH(who);
    }
    MOE_REQUIRE(fragments || L <= 256, MOE_ERR_UNSUPPORTED, "%s: row-major states are taken up to 256 positions", who);
    // row-major states come from sequences shorter than a fragment image needs
#define MOE_ATT(NKS)                                                                                            \
    (!fragments ? sru_attention_kernel<NKS, 4, false>                                                           \
     : L <= 256 ? sru_attention_kernel<NKS, 4, true>                                                            \
     : L <= 512 ? sru_attention_kernel<NKS, 8, true>                                                            \
                : sru_attention_kernel<NKS, 16, true>)
    auto kern = n == 128 ? MOE_ATT(8) : MOE_ATT(16);
#undef MOE_ATT
    const int units = ceil_div(L, ATT_QT) * B;
    hipLaunchKernelGGL(kern, dim3((int)align_up((size_t)units, 8)), dim3(ATT_THREADS), 0, st, (const bf16_t *)h,
                       (const bf16_t *)ht_ws, units, L, Lp, (bf16_t *)z);
    MOE_CHECK_LAUNCH(who);
    return MOE_OK;
}

}  // namespace moe
