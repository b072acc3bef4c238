// Router for every shape the packed bf16 kernels do not take: binary32 tensors, any expert count, any d that is a
// multiple of 8.  The router matrix is read as it lies, row-major [d, E], so no re-layout and no scratch is needed.
//
// One workgroup = 32 tokens (few binary32 ones: 16) x all experts; its wavefronts, four or more for small batches, split k, so nothing is shared and nothing waits
// until the partial sums meet in LDS at the end.  What bounds this kernel is latency (a few hundred workgroups, a
// few hundred KB each, all of it in L2 after the first reader), so the loads of U steps are in flight at once.
//
// Matrix operand.  A matrix instruction wants, per lane, consecutive k of ONE column, while the matrix has
// consecutive columns of one k.  Which expert a column index of the instruction stands for is free, so lane j of 32
// loads VEC neighbouring columns j*VEC .. +VEC-1 of each k with one wide load and uses column s of them in strip s:
//   bf16  v_mfma_f32_32x32x16_bf16, a step is 16 k (8 per lane half): 8 loads, then byte permutes pair up the k's
//   f32   v_mfma_f32_32x32x2_f32, a step is 8 k (4 per lane half, one per instruction): 4 loads, used as they are; with 16 tokens
//         v_mfma_f32_16x16x4_f32, a step is 16 k
// VEC grows with E (1, 2, 4, 8 for up to 32, 64, 128, 256 experts, as far as E's divisibility keeps the loads
// aligned); more experts than 32 * VEC are walked in groups whose logits collect in LDS.
//
// Measured (a call in a captured graph), us: 3001 tokens x 768, 64 experts, bf16 81 -> 6.2; 1500 x 512, 32 experts, f32 167 -> 5.0, against
// one wavefront per token with the experts over the lanes (a serial chain of d multiply-adds behind 2- or 4-byte loads); of it the wavefronts
// past four and the tiles of 16 tokens 7.3 -> 6.2 and 7.8 -> 5.0.
#pragma once
#include "gemm_bf16.h"

namespace moe {

constexpr int RD_BM = 32, RD_BM_F32 = 16;    // tokens per workgroup
constexpr int RD_FEW_TILES = 256;

template <bool BF16, int VEC, int NG>
struct RdLoads {
    static constexpr int KL = BF16 ? 8 : 4;                                // consecutive k per lane and step
    static constexpr int BW = BF16 ? (VEC > 1 ? VEC / 2 : 1) : VEC;        // 32-bit words per k
    uint4 a;
    uint32_t b[KL][NG][BW];
};

template <int WORDS>
__device__ __forceinline__ void rd_load_words(uint32_t (&dst)[WORDS], const void *p)
{
    if constexpr (WORDS == 1) dst[0] = *reinterpret_cast<const uint32_t *>(p);
    if constexpr (WORDS == 2) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        dst[0] = v.x;
        dst[1] = v.y;
    }
    if constexpr (WORDS >= 4) {
#pragma unroll
        for (int i = 0; i < WORDS / 4; ++i) {
            const uint4 v = reinterpret_cast<const uint4 *>(p)[i];
            dst[4 * i] = v.x;
            dst[4 * i + 1] = v.y;
            dst[4 * i + 2] = v.z;
            dst[4 * i + 3] = v.w;
        }
    }
}

// GROUPS: E > BM * VEC * NG.  NG: runs of VEC columns a lane has in a group.  BM: tokens.  NW: wavefronts, over which k is split
template <bool BF16, int VEC, int NG, bool GROUPS, int BM, int NW>
__global__ __launch_bounds__(NW * WAVE, 1) void route_direct_kernel(const void *__restrict__ xv,
                                                                       const void *__restrict__ wv,
                                                                       const float *__restrict__ bias, int T, int d,
                                                                       int E, int top_k, int renormalize,
                                                                       int32_t *__restrict__ idx,
                                                                       float *__restrict__ prob,
                                                                       float *__restrict__ logits_opt)
{
    using Loads = RdLoads<BF16, VEC, NG>;
    static_assert(BM == 32 || !BF16, "16 tokens: binary32 only");
    constexpr int KL = Loads::KL, KS = WAVE / BM * KL, ESZ = BF16 ? 2 : 4, GW = BM * VEC * NG;   // GW: columns per group
    // steps in flight: twice U with four wavefronts, U with more (16 of them have 128 registers each, and hide each other's waits)
    constexpr int U = NW > 4 ? (BM == 16 && VEC * NG <= 4 ? 8 : 4) : VEC <= 2 ? 6 : VEC == 4 ? 4 : 2;
    static_assert(GROUPS || NW * VEC <= 32, "a partial tile per wavefront fits");
    constexpr int SLOTS = GROUPS ? 1 : NW;
    constexpr int LD = (GROUPS ? MOE_MAX_EXPERTS : GW) + 4;
    __shared__ __attribute__((aligned(16))) float part[SLOTS][BM][LD];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, j = lane % BM, h = lane / BM;
    const int row0 = blockIdx.x * BM;
    const int n_steps = (d + KS - 1) / KS;
    const int s_begin = n_steps * w / NW, s_end = n_steps * (w + 1) / NW;
    const int xrow = row0 + j < T ? row0 + j : T - 1;            // rows past the batch repeat its last row
    const char *xp = (const char *)xv + (size_t)xrow * d * ESZ;
    const size_t w_stride = (size_t)E * ESZ;

    // reduction roles: thread (r, sub) of TPR threads per token
    constexpr int TPR = NW * WAVE / BM;
    const int r = tid / TPR, sub = tid % TPR;
    const int grow = row0 + r;
    const bool live = grow < T;
    constexpr int PER = GROUPS ? 1 : GW / TPR, VW = PER < 4 ? PER : 4;
    float lv[PER];                                               // this thread's logits: column col_of(i)
    auto col_of = [&](int i) { return (i / VW * TPR + sub) * VW + i % VW; };

    for (int g0 = 0; g0 < (GROUPS ? E : 1); g0 += GW) {
        const char *wp[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int col = g0 + (g * BM + j) * VEC;
            wp[g] = (const char *)wv + (size_t)(col < E ? col : 0) * ESZ;        // columns past E: any, masked below
        }
        Loads buf[NW > 4 ? 1 : 2][U];
        auto load = [&](int s, Loads &l) {
            const int ss = s < s_end ? s : s_end - 1;
            const int k = ss * KS + h * KL;
            const int kk = k < d ? k : 0;                        // lanes past the end in the last step
            l.a = *reinterpret_cast<const uint4 *>(xp + (size_t)kk * ESZ);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const char *p = wp[g] + (size_t)kk * w_stride;   // one product per run, the rest are additions
#pragma unroll
                for (int i = 0; i < KL; ++i) {
                    if constexpr (BF16 && VEC == 1)
                        l.b[i][g][0] = *reinterpret_cast<const uint16_t *>(p + i * w_stride);
                    else
                        rd_load_words<Loads::BW>(l.b[i][g], p + i * w_stride);
                }
            }
        };
        constexpr int ACC = BM * BM / WAVE, STRIPS = VEC * NG;
        typedef float acc_t __attribute__((ext_vector_type(ACC)));
        acc_t acc[STRIPS];
#pragma unroll
        for (int s = 0; s < STRIPS; ++s)
#pragma unroll
            for (int v = 0; v < ACC; ++v) acc[s][v] = 0.f;
        auto row_of = [&](int v) { return BM == 32 ? acc_row(v, lane) : 4 * h + v; };
        auto column_of = [&](int s) { return (s / VEC * BM + j) * VEC + s % VEC; };
        auto multiply = [&](int s, Loads &l) {
            if (s >= s_end) return;                              // uniform
            if ((BF16 || BM == 16) && (s + 1) * KS > d) {        // uniform: the k's past d count as zero
                const bool past = s * KS + h * KL >= d;
                if (past) l.a = make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < KL; ++i)
#pragma unroll
                    for (int q = 0; q < Loads::BW; ++q)
#pragma unroll
                        for (int g = 0; g < NG; ++g)
                            if (past) l.b[i][g][q] = 0;
            }
            if constexpr (BF16) {
#pragma unroll
                for (int c = 0; c < VEC; ++c) {
                    uint32_t f[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        f[q] = VEC == 1 ? l.b[2 * q][0][0] | (l.b[2 * q + 1][0][0] << 16)
                                        : __builtin_amdgcn_perm(l.b[2 * q + 1][0][c / 2], l.b[2 * q][0][c / 2],
                                                                (c & 1) ? 0x07060302u : 0x05040100u);
                    acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8_t, l.a), __builtin_bit_cast(bf16x8_t, make_uint4(f[0], f[1], f[2], f[3])),
                        acc[c], 0, 0, 0);
                }
            } else {
                const uint32_t a4[4] = {l.a.x, l.a.y, l.a.z, l.a.w};
#pragma unroll
                for (int i = 0; i < KL; ++i)
#pragma unroll
                    for (int c = 0; c < STRIPS; ++c) {
                        const float a = __uint_as_float(a4[i]), b = __uint_as_float(l.b[i][c / VEC][c % VEC]);
                        if constexpr (BM == 32) acc[c] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, acc[c], 0, 0, 0);
                        else acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[c], 0, 0, 0);
                    }
            }
        };
        if constexpr (NW > 4) {
            for (int s = s_begin; s < s_end; s += U) {           // uniform per wavefront
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (s + u < s_end) load(s + u, buf[0][u]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < U; ++u) multiply(s + u, buf[0][u]);
                __builtin_amdgcn_sched_barrier(0);
            }
        } else if (s_begin < s_end) {
#pragma unroll
            for (int u = 0; u < U; ++u) load(s_begin + u, buf[0][u]);
            for (int s = s_begin; s < s_end; s += 2 * U) {
                if (s + U < s_end) {
#pragma unroll
                    for (int u = 0; u < U; ++u) load(s + U + u, buf[1][u]);
                }
                __builtin_amdgcn_sched_barrier(0);               // the loads stay ahead of the matrix instructions
#pragma unroll
                for (int u = 0; u < U; ++u) multiply(s + u, buf[0][u]);
                if (s + 2 * U < s_end) {
#pragma unroll
                    for (int u = 0; u < U; ++u) load(s + 2 * U + u, buf[0][u]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < U; ++u) multiply(s + U + u, buf[1][u]);
            }
        }
        if constexpr (GROUPS) {
            // the wavefronts add their sums to the tile one after another
            for (int p = 0; p < NW; ++p) {
                if (w == p) {
#pragma unroll
                    for (int v = 0; v < ACC; ++v)
#pragma unroll
                        for (int c = 0; c < STRIPS; ++c) {
                            float *t = &part[0][row_of(v)][g0 + column_of(c)];
                            *t = p == 0 ? acc[c][v] : *t + acc[c][v];
                        }
                }
                __syncthreads();
            }
        } else {
#pragma unroll
            for (int v = 0; v < ACC; ++v)
#pragma unroll
                for (int c = 0; c < STRIPS; ++c) part[w][row_of(v)][column_of(c)] = acc[c][v];
            __syncthreads();
        }
    }

    if constexpr (GROUPS) {
        for (int c = sub; c < E; c += TPR) {
            const float t = part[0][r][c] + (bias ? bias[c] : 0.f);
            part[0][r][c] = t;                                   // read again below by this thread only
            if (logits_opt && live) logits_opt[(size_t)grow * E + c] = t;
        }
    } else {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int c = col_of(i);
            float q[SLOTS];
#pragma unroll
            for (int p = 0; p < SLOTS; ++p) q[p] = part[p][r][c];
#pragma unroll
            for (int o = 1; o < SLOTS; o *= 2)
#pragma unroll
                for (int p = 0; p + o < SLOTS; p += 2 * o) q[p] += q[p + o];
            const float t = q[0];
            lv[i] = c < E ? t + (bias ? bias[c] : 0.f) : 0.f;
            if (logits_opt && live && c < E) logits_opt[(size_t)grow * E + c] = lv[i];
        }
    }
    // f(logit, column) for every logit of this thread, columns ascending
    auto each = [&](auto f) {
        if constexpr (GROUPS) {
            for (int c = sub; c < E; c += TPR) f(part[0][r][c], c);
        } else {
#pragma unroll
            for (int i = 0; i < PER; ++i)
                if (col_of(i) < E) f(lv[i], col_of(i));
        }
    };
    float best = -INFINITY;
    int bi = 0x7fffffff;
    each([&](float t, int c) { argmax_merge(best, bi, t, c); });
    argmax_over<TPR>(best, bi);
    float z = 0.f;
    each([&](float t, int) { z += expf(t - best); });
    z = sum_over<TPR>(z);
    const bool writer = sub == 0 && live;
    if (top_k == 1) {
        if (writer) {
            idx[grow] = bi;
            prob[grow] = 1.f / z;
        }
        return;
    }
    // choice j: the largest logit after choice j-1 in the order (logit descending, id ascending)
    int ci[MOE_MAX_TOPK];
    float cw[MOE_MAX_TOPK];
    ci[0] = bi;
    cw[0] = 1.f / z;
    float pv = best, wsum = cw[0];
    int pi = bi;
#pragma unroll
    for (int q = 1; q < MOE_MAX_TOPK; ++q) {
        if (q < top_k) {
            float v = -INFINITY;
            int vi = 0x7fffffff;
            each([&](float t, int c) {
                if (t < pv || (t == pv && c > pi)) argmax_merge(v, vi, t, c);
            });
            argmax_over<TPR>(v, vi);
            ci[q] = vi;
            cw[q] = expf(v - best) / z;
            wsum += cw[q];
            pv = v;
            pi = vi;
        }
    }
    if (writer) {
#pragma unroll
        for (int q = 0; q < MOE_MAX_TOPK; ++q)
            if (q < top_k) {
                idx[(size_t)q * T + grow] = ci[q];
                prob[(size_t)q * T + grow] = renormalize ? cw[q] / wsum : cw[q];
            }
    }
}

template <bool BF16, int VEC, int NG, int BM, int NW>
static void route_direct_launch_as(const void *x, const void *w, const float *bias, int T, int d, int E, int top_k, int renormalize,
                                   int32_t *idx, float *prob, float *logits_opt, hipStream_t st)
{
    const dim3 grid(ceil_div(T, BM)), block(NW * WAVE);
    if constexpr (BM == 32 && NW == 4) {
        if (E > BM * VEC * NG) {
            hipLaunchKernelGGL((route_direct_kernel<BF16, VEC, NG, true, BM, NW>), grid, block, 0, st, x, w, bias, T, d, E, top_k,
                               renormalize, idx, prob, logits_opt);
            return;
        }
    }
    hipLaunchKernelGGL((route_direct_kernel<BF16, VEC, NG, false, BM, NW>), grid, block, 0, st, x, w, bias, T, d, E, top_k, renormalize,
                       idx, prob, logits_opt);
}

// Columns per lane: the fewest that cover E in one group, but never so many that a lane's load of VEC columns would
// not be aligned in every row (a row is E elements, so VEC has to divide E) or from the matrix' address on (the predictor's head
// is taken at any).
// Tokens and wavefronts: a batch of up to 256 tiles has a CU for each, so what counts is how long a tile takes.  16 wavefronts instead of
// four request a share of k in one go; binary32 is bound by its CU's matrix pipes where E and d are large, and 16 tokens are half the work.
// Binary32 with up to 16 experts has 32 tokens all the same, and with a deep k four wavefronts, which keep the next steps' loads in flight
// while they multiply, are ahead of 16 that do not.  us, four and 16 wavefronts: 8 experts, 4096 tokens, d = 256 6.2, 5.0; 512 7.7, 7.2; 768 9.7,
// 9.8; 2048 20.1, 23.0; 8192 59.6, 78.4; 1000 tokens, d = 1024 11.9, 11.6; 16 tokens 10.3, 9.0.
template <bool BF16>
static void route_direct_launch(const void *x, const void *w, const float *bias, int T, int d, int E, int top_k,
                                int renormalize, int32_t *idx, float *prob, float *logits_opt, hipStream_t st)
{
    constexpr int PIECE = BF16 ? 8 : 4;                          // elements of the widest load
    const size_t at = reinterpret_cast<uintptr_t>(w) / (16 / PIECE);
    auto fits = [&](int v) { return E % v == 0 && at % (v < PIECE ? v : PIECE) == 0; };
    int vec = 1;
    while (vec < 8 && 32 * vec < E && fits(2 * vec)) vec *= 2;
#define MOE_RD(V, NG, BM, NW) \
    return route_direct_launch_as<BF16, V, NG, BM, NW>(x, w, bias, T, d, E, top_k, renormalize, idx, prob, logits_opt, st)
    const bool few = ceil_div(T, RD_BM) <= RD_FEW_TILES && E <= 32 * vec && (BF16 || (E <= 16 && d <= (T <= 1024 ? 1024 : 512)));
    if constexpr (!BF16) {
        if (ceil_div(T, RD_BM_F32) <= RD_FEW_TILES && E > 16 && E <= 128 && fits(E > 32 ? 4 : 2)) {
            if (E > 64) MOE_RD(4, 2, RD_BM_F32, 8);
            if (E > 32) MOE_RD(4, 1, RD_BM_F32, 8);
            MOE_RD(2, 1, RD_BM_F32, 8);
        }
    }
    switch (vec) {
    case 1:
        if (few) MOE_RD(1, 1, RD_BM, 16);
        MOE_RD(1, 1, RD_BM, 4);
    case 2:
        if constexpr (BF16) {
            if (few) MOE_RD(2, 1, RD_BM, 16);
        }
        MOE_RD(2, 1, RD_BM, 4);
    case 4:
        if constexpr (BF16) {
            if (few) MOE_RD(4, 1, RD_BM, 8);
        }
        MOE_RD(4, 1, RD_BM, 4);
    default: MOE_RD(8, 1, RD_BM, 4);
    }
#undef MOE_RD
}

}  // namespace moe
