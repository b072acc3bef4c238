// Pieces of replica_plan shared by its own kernels and by the fused small-batch front end:
// the ballot-aggregated LDS histogram of ids and the integer allocation run by one wavefront.
#pragma once
#include "common.h"

namespace moe {

constexpr int PLAN_THREADS = 1024;
constexpr int PLAN_BATCH = 8;  // ids fetched per thread before any of them is counted

// One lane of the row of 16 to another on the data-parallel-primitive path (no trip through LDS):
// lane ^ 1, lane ^ 2, the lane 4 further, the lane 8 further (rotations inside the row).
template <int STEP>
__device__ __forceinline__ int row_exchange(int x)
{
    if (STEP == 0) return __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, false);
    if (STEP == 1) return __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, false);
    if (STEP == 2) return __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false);
    return __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false);
}

template <int STEP>
__device__ __forceinline__ long long row_exchange_ll(long long v)
{
    const unsigned lo = (unsigned)row_exchange<STEP>((int)(unsigned)v);
    const unsigned hi = (unsigned)row_exchange<STEP>((int)(unsigned)((unsigned long long)v >> 32));
    return (long long)(((unsigned long long)hi << 32) | lo);
}

// sum over the wavefront (all 64 lanes active), result in every lane: rows of 16 folded by lane
// exchanges, the four row sums added as scalars
__device__ __forceinline__ long long wave_sum_ll(long long v)
{
    v += row_exchange_ll<0>(v);
    v += row_exchange_ll<1>(v);
    v += row_exchange_ll<2>(v);
    v += row_exchange_ll<3>(v);
    long long t = 0;
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 16 * row);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)v >> 32), 16 * row);
        t += (long long)(((unsigned long long)hi << 32) | lo);
    }
    return t;
}

constexpr int PLAN_BLOCK_TOKENS = PLAN_THREADS * PLAN_BATCH;   // ids per workgroup of the partial pass

// ballot-aggregated LDS histogram of ids [t_begin, t_end)
__device__ __forceinline__ void plan_histogram(const int32_t *__restrict__ idx, int t_begin, int t_end, int E,
                                               int nbits, int *hist)
{
    const int tid = threadIdx.x, lane = tid & 63;
    for (int t0 = t_begin; t0 < t_end; t0 += PLAN_THREADS * PLAN_BATCH) {
        int eb[PLAN_BATCH];
#pragma unroll
        for (int u = 0; u < PLAN_BATCH; ++u) {
            int t = t0 + u * PLAN_THREADS + tid;
            eb[u] = t < t_end ? idx[t] : -1;
        }
#pragma unroll
        for (int u = 0; u < PLAN_BATCH; ++u) {
            int e = eb[u];
            bool valid = e >= 0 && e < E;
            unsigned long long mask = __ballot(valid);
            if (mask == 0) continue;
            for (int b = 0; b < nbits; ++b) {
                bool bit = (e >> b) & 1;
                unsigned long long bal = __ballot(bit);
                mask &= bit ? bal : ~bal;
            }
            if (valid && (mask & ((1ull << lane) - 1ull)) == 0) atomicAdd(&hist[e], __popcll(mask));
        }
    }
}

// Load per slot n / r as a binary64 quotient.  The order of two such quotients is the exact order of the
// fractions: the division is correctly rounded, so equal fractions give equal quotients, and different
// ones differ by at least 1 / (r r') > ulp(n / r) as long as n r' < 2^52 (n < 2^31, r <= 2^13 here).
__device__ __forceinline__ double load_per_slot(int n, int r) { return (double)n / (double)r; }

// candidate (ok, oe) against the best so far: the larger load per slot wins, the lower expert id among
// equals; e < 0 = no candidate
__device__ __forceinline__ void most_loaded_merge(double &bk, int &be, double ok, int oe)
{
    if (oe >= 0 && (be < 0 || ok > bk || (ok == bk && oe < be))) {
        bk = ok;
        be = oe;
    }
}

template <int STEP>
__device__ __forceinline__ double row_exchange_f64(double v)
{
    return __builtin_bit_cast(double, row_exchange_ll<STEP>(__builtin_bit_cast(long long, v)));
}

// maxima over the wavefront: rows of 16 lanes are folded by lane exchanges, the four rows as scalars
__device__ __forceinline__ int wave_max_i32(int v)
{
    auto larger = [](int a, int b) { return a > b ? a : b; };
    v = larger(v, row_exchange<0>(v));
    v = larger(v, row_exchange<1>(v));
    v = larger(v, row_exchange<2>(v));
    v = larger(v, row_exchange<3>(v));
    return larger(larger(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
                  larger(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v)
{
    auto larger = [](unsigned long long a, unsigned long long b) { return a > b ? a : b; };
    v = larger(v, (unsigned long long)row_exchange_ll<0>((long long)v));
    v = larger(v, (unsigned long long)row_exchange_ll<1>((long long)v));
    v = larger(v, (unsigned long long)row_exchange_ll<2>((long long)v));
    v = larger(v, (unsigned long long)row_exchange_ll<3>((long long)v));
    unsigned long long m = 0ull;
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 16 * row);
        const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 16 * row);
        m = larger(m, ((unsigned long long)hi << 32) | lo);
    }
    return m;
}

constexpr int PLAN_RANKED = 4;         // up to that many experts per slot left are ranked, more are served one by one

// The allocation of Algorithm 1 with the budget cap, run by ONE wavefront entirely in registers (lane l
// owns experts l, l+64, ...; sums and arg-max searches are wavefront reductions, so the hand-out of the
// slots left by the floors needs no barrier).  hist: counts per expert (LDS), n_ids: their
// sum at most.
// Writes rep[e] (LDS) and, with write_tables, the replicas / plan_counts tables.
template <int PLAN_PER_LANE>
__device__ __forceinline__ void plan_allocate_wave(const int *hist, int *rep, int n_ids, int E, int R, int C,
                                                   int policy, int32_t *__restrict__ replicas,
                                                   int32_t *__restrict__ plan_counts, bool write_tables = true)
{
    const int lane = threadIdx.x & 63;
    int n[PLAN_PER_LANE], r[PLAN_PER_LANE];
    // ceil(n / C) - 1 (n, C < 2^31: the sum fits 32 bits unsigned, a 64-bit division is a long routine)
    auto want_of = [&](int ids) {
        const unsigned slots = ((unsigned)ids + (unsigned)C - 1u) / (unsigned)C;
        return slots > 1u ? (int)(slots - 1u) : 0;
    };
    long long dsum = 0;
#pragma unroll
    for (int i = 0; i < PLAN_PER_LANE; ++i) {
        int e = lane + i * WAVE;
        n[i] = e < E ? hist[e] : 0;
        r[i] = 1;
        dsum += want_of(n[i]);
    }
    const long long D = wave_sum_ll(dsum);
    if (D <= (long long)R) {
#pragma unroll
        for (int i = 0; i < PLAN_PER_LANE; ++i) r[i] += want_of(n[i]);
    } else {
        long long left = R;
        if (policy == 0) {
            long long used = 0;
            const bool narrow = (unsigned long long)R * (unsigned long long)D < (1ull << 32);   // uniform
#pragma unroll
            for (int i = 0; i < PLAN_PER_LANE; ++i) {
                long long extra = narrow ? (long long)(((unsigned)R * (unsigned)want_of(n[i])) / (unsigned)D)
                                         : (long long)R * want_of(n[i]) / D;
                r[i] += (int)extra;
                used += extra;
            }
            left -= wave_sum_ll(used);
        } else {
            for (;;) {
                long long nw = 0;
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) nw += (long long)r[i] - 1 < want_of(n[i]);
                nw = wave_sum_ll(nw);
                if (nw == 0) break;
                long long q = left / nw;
                if (q == 0) break;
                long long given = 0;
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) {
                    long long unmet = want_of(n[i]) - ((long long)r[i] - 1);
                    if (unmet > 0) {
                        long long g = q < unmet ? q : unmet;
                        r[i] += (int)g;
                        given += g;
                    }
                }
                left -= wave_sum_ll(given);
            }
        }
        // The slots still left go to the most loaded expert per slot, one after another; many at a time where the order among them
        // cannot matter.  us of moe_plan_dispatch one by one, by steps of exact keys, now: 4096 ids, 128 experts, 16 slots 10.1, 8.9, 8.4; 1000
        // ids, 256 experts, 1 slot 6.6, 7.0, 6.7, 64 slots with half of the ids on one 12.6, 13.6, 12.0; 4096 ids, 1024 experts, 128
        // slots 59.7, 39.2, 31.2.
        if (n_ids < (1 << 24)) {
            // Counts below 2^24, exact in binary32.  Exact keys: load per slot and expert id in ONE 64-bit integer, so a fold step is an
            // unsigned maximum.  q = floor(RN(n 2^28 / r)) is monotone in n / r, equal for equal fractions,
            // and different fractions differ by 2^28 / (r r') >= 4 (r <= 2^13), so the order of the q is the
            // exact order of the fractions; the low 10 bits hold 1023 - id (lower id wins among equals);
            // 0 = no candidate (an open expert has n > C >= 1, so its q is positive).
            auto open = [&](int ids, int slots) { return (long long)slots * C < ids; };      // wants another one
            auto slot_key = [&](int i, int ids, int slots) -> unsigned long long {
                const unsigned long long q = (unsigned long long)((double)ids * 268435456.0 / (double)slots);
                return open(ids, slots) ? (q << 10) | (unsigned long long)(1023 - (lane + i * WAVE)) : 0ull;
            };
            // Several slots per step.  Let M be the largest load that any expert would have after one more slot: every load above M is
            // served before an expert's second one, so all of those get a slot at once.  The loads are taken in binary32 here, a
            // reciprocal and a product, off by less than 2^-22 of them: m is M to that, loads above m (1 + 2^-20) are above M for certain
            // ("sure"), and all that are no lower than M are above m (1 - 2^-20) ("due").  The most loaded expert is always sure: its next
            // load is at least 2^-13 of it lower, and so are the others'.
            int sure = 0;                                        // experts
            unsigned due = 0u;                                   // this lane's, a bit each
            int n_due = 0;
            bool more = left > 1;                                // the last one goes by exact keys right away
            while (more) {
                int top = 0;                                     // loads are positive: their order is that of their bits
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) {
                    const int bits = __float_as_int((float)n[i] * __builtin_amdgcn_rcpf((float)(r[i] + 1)));
                    top = open(n[i], r[i] + 1) && bits > top ? bits : top;
                }
                const float m = __int_as_float(wave_max_i32(top)), hi = m * (1.f + 0x1p-20f), lo = m * (1.f - 0x1p-20f);
                unsigned won = 0u;
                sure = n_due = 0;
                due = 0u;
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) {
                    const float load = open(n[i], r[i]) ? (float)n[i] * __builtin_amdgcn_rcpf((float)r[i]) : 0.f;
                    sure += __popcll(__ballot(load > hi));
                    n_due += __popcll(__ballot(load > lo));
                    won |= load > hi ? 1u << i : 0u;
                    due |= load > lo ? 1u << i : 0u;
                }
                if (n_due > left) break;
                if (sure == 0) left = 0;                         // nobody is open
                more = left > sure;
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) r[i] += (won >> i) & 1u;
                left -= sure;
            }
            if (left > 0) {                                      // not enough for all that are due: exact keys
                unsigned long long key[PLAN_PER_LANE];
#pragma unroll
                for (int i = 0; i < PLAN_PER_LANE; ++i) key[i] = slot_key(i, n[i], r[i]);
                if (sure > left && n_due <= PLAN_RANKED * left) {
                    // one each for the largest keys of those due: the rank of every key among them
                    int rank[PLAN_PER_LANE];
#pragma unroll
                    for (int i = 0; i < PLAN_PER_LANE; ++i) rank[i] = 0;
#pragma unroll
                    for (int i = 0; i < PLAN_PER_LANE; ++i)
                        for (unsigned long long w = __ballot((due >> i) & 1u); w; w &= w - 1) {
                            const int l = __builtin_ctzll(w);    // uniform
                            const unsigned lo32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)key[i], l);
                            const unsigned hi32 = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(key[i] >> 32), l);
                            const unsigned long long k = ((unsigned long long)hi32 << 32) | lo32;
#pragma unroll
                            for (int q = 0; q < PLAN_PER_LANE; ++q) rank[q] += k > key[q];
                        }
#pragma unroll
                    for (int i = 0; i < PLAN_PER_LANE; ++i) r[i] += ((due >> i) & 1u) && rank[i] < left;
                } else {
                    for (; left > 0; --left) {                   // one by one; a key is one expert's: it holds the id
                        unsigned long long m = 0ull;
#pragma unroll
                        for (int i = 0; i < PLAN_PER_LANE; ++i) m = key[i] > m ? key[i] : m;
                        m = wave_max_u64(m);
                        if (m == 0ull) break;                    // nobody is open
#pragma unroll
                        for (int i = 0; i < PLAN_PER_LANE; ++i)
                            if (key[i] == m) {
                                r[i] += 1;
                                key[i] = slot_key(i, n[i], r[i]);
                            }
                    }
                }
            }
        } else {
        double key[PLAN_PER_LANE];
#pragma unroll
        for (int i = 0; i < PLAN_PER_LANE; ++i) key[i] = load_per_slot(n[i], r[i]);
        while (left > 0) {
            double bk = 0.0;
            int be = -1;
#pragma unroll
            for (int i = 0; i < PLAN_PER_LANE; ++i) {
                const bool open = (long long)r[i] * C < n[i];
                most_loaded_merge(bk, be, key[i], open ? lane + i * WAVE : -1);   // ascending ids inside a lane
            }
            most_loaded_merge(bk, be, row_exchange_f64<0>(bk), row_exchange<0>(be));
            most_loaded_merge(bk, be, row_exchange_f64<1>(bk), row_exchange<1>(be));
            most_loaded_merge(bk, be, row_exchange_f64<2>(bk), row_exchange<2>(be));
            most_loaded_merge(bk, be, row_exchange_f64<3>(bk), row_exchange<3>(be));
            {
                const long long kb = __builtin_bit_cast(long long, bk);
                double sk = 0.0;
                int se = -1;
#pragma unroll
                for (int row = 0; row < 4; ++row) {
                    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)kb, 16 * row);
                    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)kb >> 32), 16 * row);
                    most_loaded_merge(sk, se, __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo),
                                      __builtin_amdgcn_readlane(be, 16 * row));
                }
                be = se;
            }
            if (be < 0) break;
#pragma unroll
            for (int i = 0; i < PLAN_PER_LANE; ++i)
                if (be == lane + i * WAVE) {
                    r[i] += 1;
                    key[i] = load_per_slot(n[i], r[i]);
                }
            left -= 1;
        }
        }
    }
#pragma unroll
    for (int i = 0; i < PLAN_PER_LANE; ++i) {
        int e = lane + i * WAVE;
        if (e < E) {
            rep[e] = r[i];
            if (write_tables) {
                replicas[e] = r[i];
                plan_counts[e] = n[i];
            }
        }
    }
}

}  // namespace moe
