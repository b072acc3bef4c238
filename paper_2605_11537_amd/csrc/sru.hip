// sru_predict: SRU stack + linear head + argmax, the expert predictor.
//
// Per layer: (1) the concatenated weight [n_in, k*n_h] is re-laid into the packed image the MFMA B
// operand wants (small, into the workspace; skipped when the weights arrive packed, see
// sru_weights.w_layout); (2) one matrix-core product U = X * [W | W_f | W_r | (W_h)] for all B*L
// tokens at once (the part of the SRU that is parallel over time); (3) the recurrence.  The gates
// depend on the input only, so c_t = f_t c_{t-1} + (1-f_t) x'_t is a linear recurrence in c: a
// workgroup takes a few channels of one sequence and cuts the time axis into 64 chunks; every thread
// first composes its chunk into (A, B) with c_out = A c_in + B, the 64 chunk maps of a channel are
// composed by a scan, and each thread then re-runs its chunk from its true carry-in and writes h_t.
// For sequences of up to 1024 positions steps (2) and (3) are one kernel per layer with the projections
// kept in LDS (sru_layer_fused_kernel below); the two-kernel form (sru_proj_kernel, sru_scan_kernel)
// serves longer sequences, and those of over 512 positions where it is the faster one (sru_forms.h).  The head is a router-shaped product + argmax and reuses the router's kernel.
#include "gemm_bf16.h"
#include "route.h"
#include "sru_forms.h"

namespace moe {

constexpr int SRU_CHUNKS = 64;     // time chunks per sequence
constexpr int SRU_CHANNELS = 16;   // channels per workgroup (SRU_CHUNKS * SRU_CHANNELS = 1024 threads)

// U[T, N] (fp32) = X[T, K] (bf16) * packed W
__global__ __launch_bounds__(GEMM_THREADS) void sru_proj_kernel(const bf16_t *__restrict__ X,
                                                                const bf16_t *__restrict__ Wp, int T, int K, int N,
                                                                float *__restrict__ U)
{
    __shared__ __attribute__((aligned(16))) bf16_t lds[gemm_lds_elems<2, 64>()];
    const int n_nt = N / 128;
    const int mt = blockIdx.x / n_nt, nt = blockIdx.x - mt * n_nt;
    const int row0 = mt * 64;
    const int nrows = T - row0 < 64 ? T - row0 : 64;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    f32x16_t acc[2][1];
    zero_acc<2, 1>(acc);
    gemm_tile_bf16<2, 1, 64>(X + (size_t)row0 * K, K, nrows, Wp, nt * 128, K, lds, acc);
    const int col = nt * 128 + w * 32 + (lane & 31);
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            int r = mb * 32 + acc_row(v, lane);
            if (r < nrows) U[(size_t)(row0 + r) * N + col] = acc[mb][0][v];
        }
}

// 1 / x for finite x >= 1: the hardware reciprocal and one Newton step (the full division is ten instructions, and the gates
// are most of what a layer's recurrence issues)
__device__ __forceinline__ float recip_(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.f), r);
}
// binary32 with the hardware exponential: a few ulp, far inside the bf16 rounding of h, down to the smallest normal number.  An
// infinite denominator is held at the largest finite one (sigmoid 0 or below 2^-126); the comparison leaves a NaN a NaN.
__device__ __forceinline__ float sigmoidf_(float v)
{
    const float x = 1.f + __expf(-v);
    return recip_(x > 3.402823466e38f ? 3.402823466e38f : x);
}
// The same exponential and reciprocal: an absolute error of about 1e-7.  1 - 2 / (1 + e^2a) cancels for small |v| (relative error 1.4e-3 at
// 1e-5, 5e-2 at 1e-6), which the bf16 rounding of h only covers beside a highway or other states of ordinary size.
__device__ __forceinline__ float tanhf_(float v)
{
    float a = fminf(fabsf(v), 15.f);
    float t = fmaf(-2.f, recip_(1.f + __expf(2.f * a)), 1.f);
    return copysignf(t, v);
}

// 16-byte piece of position t, channels 8g .. 8g+7, in the fragment image of a sequence's states (n channels, blocks of 32
// positions; fragment (block, 16 channels) = 64 lanes x 16 bytes, the lane order of the matrix instruction's operand)
__device__ __forceinline__ size_t packed_piece(int seq, int n_blocks, int n, int t, int g)
{
    return (((size_t)seq * n_blocks + (t >> 5)) * (n >> 4) + (g >> 1)) * 64 + (g & 1) * 32 + (t & 31);
}

// grid (n_h/16, B); block = 16 channels x 64 time chunks.  Phase 1: every thread composes its
// chunk into (A, B) with c_out = A*c_in + B.  Phase 2: one wavefront per channel composes the 64
// chunk maps by a scan.  Phase 3: every thread re-runs its chunk from its true carry-in and writes h_t.
// CL > 0: a chunk holds at most CL steps and the thread keeps all its inputs in registers -- every load of
// the kernel is issued up front, one memory round trip instead of four (U was written by other XCDs a
// moment ago, so each exposed round trip is a miss in this XCD's L2).  CL = 0: any chunk length, the
// inputs are streamed twice.
template <int CL>
__global__ __launch_bounds__(SRU_CHUNKS * SRU_CHANNELS) void sru_scan_kernel(
    const float *__restrict__ U, const bf16_t *__restrict__ x_in, int L, int n_h, int k,
    const float *__restrict__ b_f, const float *__restrict__ b_r, int packed_out, bf16_t *__restrict__ h_out)
{
    __shared__ float carry_a[SRU_CHUNKS][SRU_CHANNELS], carry_b[SRU_CHUNKS][SRU_CHANNELS];
    const int ch = threadIdx.x & (SRU_CHANNELS - 1), q = threadIdx.x / SRU_CHANNELS;
    const int j = blockIdx.x * SRU_CHANNELS + ch;
    const int b = blockIdx.y;
    const int ncol = k * n_h;
    const int cl = (L + SRU_CHUNKS - 1) / SRU_CHUNKS;
    const int t0 = q * cl < L ? q * cl : L, t1 = (t0 + cl < L) ? t0 + cl : L;
    const float bf = b_f ? b_f[j] : 0.f, br = b_r ? b_r[j] : 0.f;
    const float *u = U + (size_t)b * L * ncol + j;
    const bf16_t *xi = x_in + (size_t)b * L * n_h + j;   // only read when k == 3 (n_in == n_h)
    // row-major states, or (up to 1024 positions) the fragment image that the one-kernel layer reads (packed_piece: channel j is element j % 8 of its piece)
    const bool image = CL > 0 && packed_out;
    bf16_t *ho = image ? h_out + packed_piece(b, (L + 31) >> 5, n_h, 0, j >> 3) * 8 + (j & 7) : h_out + (size_t)b * L * n_h + j;
    auto place = [&](int t) { return image ? (size_t)(t >> 5) * n_h * 32 + (t & 31) * 8 : (size_t)t * n_h; };

    constexpr int NR = CL > 0 ? CL : 1;
    float ux[NR], uf[NR], ur[NR], uh[NR];
    if (CL > 0) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int t = t0 + i;
            const bool ok = t < t1;
            const float *ut = u + (size_t)(ok ? t : t0) * ncol;
            ux[i] = ok ? ut[0] : 0.f;
            uf[i] = ok ? ut[n_h] : 0.f;
            ur[i] = ok ? ut[2 * n_h] : 0.f;
            uh[i] = !ok ? 0.f : (k == 4 ? ut[3 * n_h] : bf16_to_f32(xi[(size_t)t * n_h]));
        }
    }

    float a = 1.f, c = 0.f;
    if (CL > 0) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (t0 + i < t1) {
                const float f = sigmoidf_(uf[i] + bf);
                uf[i] = f;                               // the gate itself from here on
                a *= f;
                c = f * c + (1.f - f) * ux[i];
            }
    } else {
#pragma unroll 4
        for (int t = t0; t < t1; ++t) {
            const float *ut = u + (size_t)t * ncol;
            float f = sigmoidf_(ut[n_h] + bf);
            a *= f;
            c = f * c + (1.f - f) * ut[0];
        }
    }
    carry_a[q][ch] = a;
    carry_b[q][ch] = c;
    __syncthreads();
    // Carry-in of every chunk, in place (carry_b[p] <- state entering chunk p): the 64 chunk maps
    // c -> a c + b of a channel are composed by an inclusive scan across the 64 lanes of one wavefront
    // (wavefront w takes channel w; six doubling steps instead of a serial chain of 64 LDS round trips,
    // which was ~40 % of this kernel's time)
    {
        const int lane = threadIdx.x & 63, sc = threadIdx.x >> 6;      // lane = chunk, sc = channel
        float pa = carry_a[lane][sc], pb = carry_b[lane][sc];
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const float qa = __shfl_up(pa, o, 64), qb = __shfl_up(pb, o, 64);   // the map of the chunks before
            if (lane >= o) {
                pb = pa * qb + pb;       // (this) o (earlier): c -> pa (qa c + qb) + pb
                pa = pa * qa;
            }
        }
        // state after chunks 0..lane from c = 0 is pb; chunk lane + 1 starts from it
        const float into_next = pb;
        const float mine = __shfl_up(into_next, 1, 64);
        __syncthreads();                 // every (a, b) has been read before any carry is overwritten
        carry_b[lane][sc] = lane == 0 ? 0.f : mine;
    }
    __syncthreads();
    c = carry_b[q][ch];

    if (CL > 0) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (t0 + i < t1) {
                const float f = uf[i];
                const float r = sigmoidf_(ur[i] + br);
                c = f * c + (1.f - f) * ux[i];
                ho[place(t0 + i)] = f32_to_bf16(r * tanhf_(c) + (1.f - r) * uh[i]);
            }
        return;
    }
#pragma unroll 4
    for (int t = t0; t < t1; ++t) {
        const float *ut = u + (size_t)t * ncol;
        float f = sigmoidf_(ut[n_h] + bf);
        float r = sigmoidf_(ut[2 * n_h] + br);
        c = f * c + (1.f - f) * ut[0];
        float hw = k == 4 ? ut[3 * n_h] : bf16_to_f32(xi[(size_t)t * n_h]);
        ho[place(t)] = f32_to_bf16(r * tanhf_(c) + (1.f - r) * hw);
    }
}

// ------------------------------------------------------------------ one SRU layer in one kernel (L <= 1024)
// Workgroup (channel block cb of 8 channels, sequence b): the projections of ITS 8 channels for all L
// positions -- 32 columns of [W | W_f | W_r | (W_h)], one matrix-core column block, gathered from the packed
// image piece by piece -- land in LDS (L x 32 binary32), and the recurrence runs from there: 64 time chunks
// x 8 channels, chunk maps composed by a scan (inside a wavefront by lane exchanges, over the eight wavefronts through
// LDS), every chunk re-run from its true carry-in.  The projections never go to memory (the two-kernel form writes and
// re-reads 3-4 binary32 values per position and channel, and its scan was bound by what one CU can fetch), there is one
// launch per layer instead of two, and B * n_h / 8 workgroups cover the chip at 8 sequences x 256 channels.
// Between layers the states are kept as matrix-core fragments (packed_piece below): a layer's output piece, 8 channels of one
// position, is 16 bytes of such a fragment, so the 32 positions of a block leave as a run of 512 bytes, and the next layer's
// operand load is 1 KB of consecutive memory, straight into registers.  Only the first layer's input (the caller's row-major
// embeddings) goes through a wavefront-private LDS transposition, which costs as much LDS time per k as the loads take.  All loads are unconditional (rows past the sequence repeat its last
// row, columns past the gates repeat the first's; neither is used), so that the waits of the chunk pipeline are counts:
// with conditional ones every chunk waited for the chunk just requested.
// Up to 256 positions a workgroup is small enough for two on a CU (128 registers, 37 KB), runs as many recurrence steps as it
// has, and only the wavefronts that have rows load any: with one per CU, four steps and all eight wavefronts loading, 64 sequences of
// 7, 256 -> 256, took 45.7 us with the head where the kernel before took 38.6, now 18; 16 x 16: 15.5, 13.8, now 9.1; 1 x 1: 10.2, 9.2,
// now 7.6.
// Measured per layer at 8 x 512, 256 -> 256, in a predictor of ten: 12.4 -> 9.0 us (8.0 .. 8.3 at best); 5 x 777, 768 -> 256 and 256 -> 256, both layers, packing and
// head: 42 us against 56 us with projection and scan kernels.
constexpr int FUS_THREADS = 512;       // 8 wavefronts: 2 per SIMD, so one's loads fly under the other's work
constexpr int FUS_WAVES = FUS_THREADS / 64;
constexpr int FUS_CHUNKS = FUS_THREADS / FUS_CH;   // 64 time chunks per sequence
constexpr int FUS_LDU = 33;            // row stride of the LDS tile, binary32 elements

// Row-major embeddings [B*L, K] -> fragment image (positions past a sequence repeat its last).  32 positions x 64 channels per
// workgroup: whole lines in, 4 KB runs out, written on the XCD whose layer workgroups read them (8 x 1024, 512 -> 256, with the layer and the head: 32.3
// -> 29.0 us).
__global__ __launch_bounds__(256) void sru_pack_input_kernel(const uint4 *__restrict__ x, int n_units, int L, int K,
                                                             uint4 *__restrict__ image)
{
    __shared__ uint4 buf[256];
    const int tid = threadIdx.x, r = tid >> 3, g = tid & 7, n_blocks = (L + 31) >> 5;
    const int unit = xcd_remap(blockIdx.x, n_units);
    if (unit < 0) return;
    const int row_blk = unit / (K >> 6), kc = unit - row_blk * (K >> 6), b = row_blk / n_blocks, blk = row_blk - b * n_blocks;
    const int t = blk * 32 + r < L ? blk * 32 + r : L - 1;
    buf[(g >> 1) * 64 + (g & 1) * 32 + r] = x[((size_t)b * L + t) * (K >> 3) + kc * 8 + g];
    __syncthreads();
    image[((size_t)b * n_blocks + blk) * (K >> 4) * 64 + kc * 256 + tid] = buf[tid];
}

// NRB: 32-row blocks per wavefront, L <= 256 * NRB.  PIN: X is a fragment image (else row-major); packed_out: so is h_out.
// WF > 0: the weight fragments (K / 16 <= 8 * WF of them) are fetched once per workgroup, WF per wavefront, and read from LDS;
// loaded by every wavefront for itself they are a third of what the CU's load path carries (45 bytes per clock, the bound of the
// product here).
// DEALT: see below; a build of its own, for every argument and instruction in front of the first load is one of each layer (as arguments: a predictor of ten
// layers 113 -> 114 us).
template <int NRB, bool PIN, int WF, bool DEALT>
__global__ __launch_bounds__(FUS_THREADS, NRB == 1 ? 4 : 1) void sru_layer_fused_kernel(const bf16_t *__restrict__ X,
                                                                         const bf16_t *__restrict__ Wp, int L, int K,
                                                                         int n_h, int kgates,
                                                                         const float *__restrict__ b_f,
                                                                         const float *__restrict__ b_r, int packed_out,
                                                                         bf16_t *__restrict__ h_out,
                                                                         bf16_t *__restrict__ ht_out)
{
    constexpr int MAX_L = 256 * NRB;
    constexpr int KC = NRB <= 2 ? 64 : 32;             // k per register buffer: a whole line per row, or half of one for room
    constexpr int LDA = KC + 8;
    constexpr int SB = NRB < 2 ? NRB : 2;              // row blocks a wavefront stages at a time
    // the L x 32 tile of projections; during the product, the weight fragments and the wavefronts' staging pieces for the token rows
    constexpr int TILE_FLOATS = MAX_L * FUS_LDU, W_FLOATS = WF * FUS_WAVES * 256;
    constexpr int STAGE_FLOATS = W_FLOATS + (PIN ? 0 : FUS_WAVES * SB * 32 * LDA / 2);
    __shared__ __attribute__((aligned(16))) float u_lds[TILE_FLOATS > STAGE_FLOATS ? TILE_FLOATS : STAGE_FLOATS];
    __shared__ float wave_a[FUS_WAVES][FUS_CH], wave_b[FUS_WAVES][FUS_CH];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroup i runs on XCD i % 8.  All channel blocks of a sequence read the same token rows, written a moment ago by the layer before: 8
    // contiguous ranges of the (sequence, channel block) pairs, one per XCD, so that an XCD's L2 fetches about 1/8 of the rows instead of all
    // of them, and mostly those it wrote (n_h / 8 is a multiple of 16, the ranges are equal).  DEALT: the channel blocks of a sequence go to all
    // XCDs in turn, so that an L2 holds 1/8 of the weights instead (sru_deals_channels).  With the channel blocks of a sequence dealt to all XCDs
    // where the sequences are no multiple of 8, us: 12 x 512, 256 -> 256, four layers 76.0, now 67.8; 5 x 512, 768 -> 256, two 30.5, 28.9.
    int cb, b;
    {
        const int ncb = n_h / FUS_CH, at = DEALT ? blockIdx.x : (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
        b = at / ncb;
        cb = at - b * ncb;
    }
    const int KG = K >> 3;
    typedef unsigned u32x4s_t __attribute__((ext_vector_type(4)));
    const bf16_t *Xs = X + (size_t)b * L * K;
    const u32x4s_t *Xp = reinterpret_cast<const u32x4s_t *>(X);
    const int n_blocks = (L + 31) >> 5;
    const int ch = tid & (FUS_CH - 1), q = tid / FUS_CH;      // recurrence roles: thread = (chunk q, channel ch)
    const int j = cb * FUS_CH + ch;
    const float bf = b_f ? b_f[j] : 0.f, br = b_r ? b_r[j] : 0.f;
    // highway input when the widths are equal (K == n_h): this workgroup's 8 channels of row tid (and tid + 512)
    constexpr int HROWS = (MAX_L + FUS_THREADS - 1) / FUS_THREADS;
    u32x4s_t hw_in[HROWS];
    if (kgates == 3) {
#pragma unroll
        for (int i = 0; i < HROWS; ++i) {
            int t = tid + i * FUS_THREADS;
            t = t < L ? t : L - 1;
            hw_in[i] = PIN ? Xp[packed_piece(b, n_blocks, K, t, cb)]
                           : *reinterpret_cast<const u32x4s_t *>(Xs + (size_t)t * K + cb * FUS_CH);
        }
    }
    // ---- projections: U[t][c], c = gate * 8 + channel
    {
        const int r = lane & 31;
        f32x16_t acc[NRB][1];
        zero_acc<NRB, 1>(acc);
        // One body per number of row blocks a wavefront has.  With NRB for everybody, the blocks that a wavefront does not have were up to a third of
        // the loads: 6 x 600, 256 -> 256, four layers with the head, 57.6 -> 47.4 us (with the recurrence's steps below); 8 x 300, 768 -> 256, one
        // layer 19.5 -> 16.3; 5 x 777, 768 -> 256, two layers 46.9 -> 42.4.
        auto product = [&](auto BLOCKS) {
            constexpr int MB = decltype(BLOCKS)::value;
            // Token rows: a wavefront fetches its own row blocks in whole 128-byte lines (8 lanes per row, 8 rows
            // per load; half lines for the longest sequences), turns them into A fragments through a private piece of LDS (row stride 72 elements, no
            // barrier: LDS operations of one wavefront execute in order).  A lane
            // loading its fragment straight from memory touches 32 bytes of 32 different lines per load, and
            // the kernel was bound by those transactions.
            bf16_t *stage = reinterpret_cast<bf16_t *>(u_lds + W_FLOATS) + (size_t)w * (SB * 32 * LDA);
            u32x4s_t *w_lds = reinterpret_cast<u32x4s_t *>(u_lds);
            const int kh = lane >> 5;
            constexpr int PPR = KC / 8, RPL = 64 / PPR, NSB = 32 / RPL;      // pieces per row, rows per load, loads per row block
            const int lrow = lane / PPR, lpiece = lane % PPR;
            // this lane's pieces of its rows, elements from the sequence's first; or the first fragment of its row blocks
            unsigned a_off[MB][NSB];
            const u32x4s_t *a_frag[MB];
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int sb = 0; sb < NSB; ++sb) {
                    const int t = (w + FUS_WAVES * i) * 32 + sb * RPL + lrow;   // row blocks dealt to the eight wavefronts in turn
                    a_off[i][sb] = (unsigned)(t < L ? t : L - 1) * K + lpiece * 8;
                }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int blk = w + FUS_WAVES * i < n_blocks ? w + FUS_WAVES * i : n_blocks - 1;
                a_frag[i] = Xp + ((size_t)b * n_blocks + blk) * (K >> 4) * 64;
            }
            const int gate = r >> 3 < kgates ? r >> 3 : 0;
            const int col = gate * n_h + cb * FUS_CH + (r & 7);
            const u32x4s_t *b_ptr = reinterpret_cast<const u32x4s_t *>(Wp) + ((size_t)(col >> 5) * KG + kh) * 32 + (col & 31);
            constexpr int KS = KC / 16;
            // Chunks in flight, of which D - 1 are asked for past the end.  Short row-major sequences: two, which leaves room for a second
            // workgroup per CU (see the launch bounds).  Narrow first layers have 1 .. 8 chunks, and the other wavefront's loads to hide
            // behind: 2 x 300, 64 -> 128, with the head, three, two, one chunk: 10.8, 10.5, 9.9 us; 16 x 1024, 256 -> 256: 46.1, 44.3, 43.5.
            constexpr int D = PIN ? 3 : WF == 2 ? 1 : NRB == 1 ? 2 : 3;
            constexpr int AR = PIN ? KS : NSB;             // 16-byte pieces per lane, row block and chunk (the same number)
            u32x4s_t ga[D][MB][AR], fb[WF ? 1 : D][KS], wf[WF ? WF : 1];
            const int nkc = K / KC;
            auto load = [&](int kc, int buf) {
                const int k0 = (kc < nkc ? kc : nkc - 1) * KC;         // past the end: a harmless re-read
                if constexpr (WF == 0) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) fb[buf][ks] = b_ptr[(size_t)((k0 >> 3) + ks * 2) * 32];
                }
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int sb = 0; sb < AR; ++sb)
                        ga[buf][i][sb] = PIN ? a_frag[i][((k0 >> 4) + sb) * 64 + lane]
                                             : *reinterpret_cast<const u32x4s_t *>(Xs + k0 + a_off[i][sb]);
                __builtin_amdgcn_sched_barrier(0);
            };
            auto compute = [&](int kc, int buf) {
                const int fbuf = WF ? 0 : buf;
                if constexpr (WF > 0) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) fb[0][ks] = w_lds[(kc * KS + ks) * 64 + lane];
                }
                if constexpr (PIN) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int i = 0; i < MB; ++i)
                            acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ga[buf][i][ks]),
                                                                                __builtin_bit_cast(bf16x8_t, fb[fbuf][ks]),
                                                                                acc[i][0], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    return;
                }
#pragma unroll
                for (int i0 = 0; i0 < MB; i0 += SB) {
#pragma unroll
                    for (int i = 0; i < SB && i0 + i < MB; ++i)
#pragma unroll
                        for (int sb = 0; sb < NSB; ++sb)
                            *reinterpret_cast<u32x4s_t *>(stage + (i * 32 + sb * RPL + lrow) * LDA + lpiece * 8) = ga[buf][i0 + i][sb];
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                        for (int i = 0; i < SB && i0 + i < MB; ++i) {
                            const u32x4s_t av = *reinterpret_cast<const u32x4s_t *>(stage + (i * 32 + r) * LDA + ks * 16 + kh * 8);
                            acc[i0 + i][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, av),
                                                                                     __builtin_bit_cast(bf16x8_t, fb[fbuf][ks]),
                                                                                     acc[i0 + i][0], 0, 0, 0);
                        }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (WF > 0) {
                const int n_frag = K >> 4;
#pragma unroll
                for (int i = 0; i < WF; ++i) {
                    const int fr = w + FUS_WAVES * i < n_frag ? w + FUS_WAVES * i : n_frag - 1;
                    wf[i] = b_ptr[(size_t)(fr * 2) * 32];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // A wavefront whose first row block lies past the sequence multiplies nothing: eight of them loaded the same rows at 7 positions.
            // (Where weights are shared the loads stay unconditional, the wait for the weights is a count over them.)
            const bool rows = WF > 0 || w * 32 < L;
            if (rows) {
#pragma unroll
                for (int d = 0; d < D; ++d) load(d, d);
            }
            if constexpr (WF > 0) {
#pragma unroll
                for (int i = 0; i < WF; ++i) w_lds[(w + FUS_WAVES * i) * 64 + lane] = wf[i];
                // (one __syncthreads between two halves of the body keeps the rows in flight across a join: 178 registers for 148 at best, up to 85
                // spilled)
                barrier_anywhere();
            }
            const int n_chunks = rows ? nkc : 0;
            int kc = 0;
            for (; kc + D < n_chunks; kc += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    compute(kc + d, d);
                    load(kc + D + d, d);
                }
            }
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (kc + d < n_chunks) compute(kc + d, d); // uniform
        };
        using std::integral_constant;
        const int n_own = (n_blocks - w + FUS_WAVES - 1) / FUS_WAVES;            // NRB / 2 and more
        if (NRB == 1 || n_own == NRB) product(integral_constant<int, NRB>{});
        else if (NRB == 4 && n_own == 3) product(integral_constant<int, NRB == 4 ? 3 : NRB>{});
        else product(integral_constant<int, (NRB > 1 ? NRB / 2 : 1)>{});
        __syncthreads();           // the staging pieces alias the tile written next
        if (r < kgates * FUS_CH) {
#pragma unroll
            for (int i = 0; i < NRB; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) u_lds[((w + FUS_WAVES * i) * 32 + acc_row(v, lane)) * FUS_LDU + r] = acc[i][0][v];
        }
        if (kgates == 3) {         // the highway input takes the place of the fourth gate
#pragma unroll
            for (int i = 0; i < HROWS; ++i) {
                const int t = tid + i * FUS_THREADS;
                if (t < MAX_L) {
                    float *ut = u_lds + t * FUS_LDU + 3 * FUS_CH;
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        ut[2 * c] = __uint_as_float(hw_in[i][c] << 16);
                        ut[2 * c + 1] = __uint_as_float(hw_in[i][c] & 0xffff0000u);
                    }
                }
            }
        }
    }
    __syncthreads();

    // ---- recurrence: chunk q holds positions q*cl .. ; past the end of the sequence a step is the identity
    const int cl = (L + FUS_CHUNKS - 1) / FUS_CHUNKS, t0 = q * cl;
    bf16_t *h_lds = reinterpret_cast<bf16_t *>(u_lds);
    auto recurrence = [&](auto STEPS) {                // of up to STEPS positions per chunk
        constexpr int CL = decltype(STEPS)::value;
        float f[CL], g[CL], r[CL], hw[CL];
#pragma unroll
        for (int i = 0; i < CL; ++i) {
            const int t = t0 + i;
            const float *ut = u_lds + (t < MAX_L ? t : MAX_L - 1) * FUS_LDU + ch;
            g[i] = ut[0];
            f[i] = ut[FUS_CH];
            r[i] = ut[2 * FUS_CH];
            hw[i] = ut[3 * FUS_CH];
        }
        float a = 1.f, c = 0.f;
#pragma unroll
        for (int i = 0; i < CL; ++i) {
            const bool in = i < cl && t0 + i < L;
            f[i] = in ? sigmoidf_(f[i] + bf) : 1.f;
            g[i] = in ? (1.f - f[i]) * g[i] : 0.f;
            r[i] = sigmoidf_(r[i] + br);
            a *= f[i];
            c = f[i] * c + g[i];
        }
        // Inclusive scan of the chunk maps c -> a c + b.  A wavefront holds 8 neighbouring chunks x 8 channels: three
        // doubling steps over lanes 8, 16, 32 apart; then the eight wavefronts' totals, composed by every thread for itself.
#pragma unroll
        for (int o = FUS_CH; o < 64; o <<= 1) {
            const float qa = __shfl_up(a, o, 64), qb = __shfl_up(c, o, 64);
            if (lane >= o) {
                c = a * qb + c;                                // (this) after (earlier)
                a = a * qa;
            }
        }
        if (lane >= 64 - FUS_CH) {
            wave_a[w][ch] = a;
            wave_b[w][ch] = c;
        }
        // the map of the chunks before this one, inside the wavefront
        float pa = __shfl_up(a, FUS_CH, 64), pb = __shfl_up(c, FUS_CH, 64);
        if (lane < FUS_CH) {
            pa = 1.f;
            pb = 0.f;
        }
        __syncthreads();               // also: every projection has been read, the tile is free for the output rows
        float cin = 0.f;
#pragma unroll
        for (int i = 0; i < FUS_WAVES - 1; ++i)
            if (i < w) cin = wave_a[i][ch] * cin + wave_b[i][ch];
        c = pa * cin + pb;

        // h of 8 channels makes a 16-byte piece per position: through LDS, one store per row instead of eight of 2 bytes
#pragma unroll
        for (int i = 0; i < CL; ++i) {
            c = f[i] * c + g[i];
            if (i < cl && t0 + i < L) h_lds[(t0 + i) * FUS_CH + ch] = f32_to_bf16(r[i] * tanhf_(c) + (1.f - r[i]) * hw[i]);
        }
    };
    // the steps that the chunks have, to the next even number (a step past the chunk costs as much as one inside)
    using std::integral_constant;
    if (NRB == 4) {
        if (cl > 14) recurrence(integral_constant<int, NRB == 4 ? 16 : 1>{});
        else if (cl > 12) recurrence(integral_constant<int, NRB == 4 ? 14 : 1>{});
        else if (cl > 10) recurrence(integral_constant<int, NRB == 4 ? 12 : 1>{});
        else recurrence(integral_constant<int, NRB == 4 ? 10 : 1>{});
    } else if (NRB == 2) {
        if (cl > 6) recurrence(integral_constant<int, NRB == 2 ? 8 : 1>{});
        else recurrence(integral_constant<int, NRB == 2 ? 6 : 1>{});
    }
    else if (cl == 1) recurrence(integral_constant<int, 1>{});
    else if (cl == 2) recurrence(integral_constant<int, 2>{});
    else recurrence(integral_constant<int, 4>{});
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HROWS; ++i) {
        const int t = tid + i * FUS_THREADS;
        if (t < L) {
            u32x4s_t *dst = packed_out ? reinterpret_cast<u32x4s_t *>(h_out) + packed_piece(b, n_blocks, n_h, t, cb)
                                       : reinterpret_cast<u32x4s_t *>(h_out + ((size_t)b * L + t) * n_h + cb * FUS_CH);
            *dst = *reinterpret_cast<const u32x4s_t *>(h_lds + t * FUS_CH);
        }
    }
    // In front of the attention, also the packed image of the states as a (positions x channels) matrix (piece: 8 consecutive
    // positions of one channel, positions past the sequence zero).
    if (ht_out) {
        const int n_groups = (L + 15) / 16 * 2;
        u32x4s_t *ht = reinterpret_cast<u32x4s_t *>(ht_out) + (size_t)b * (n_h >> 5) * n_groups * 32;
        const int f = cb * FUS_CH + ch;
        for (int gr = q; gr < n_groups; gr += FUS_CHUNKS) {
            u32x4s_t v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = gr * 8 + 2 * i;
                const uint32_t lo = t < L ? h_lds[t * FUS_CH + ch] : 0, hi = t + 1 < L ? h_lds[(t + 1) * FUS_CH + ch] : 0;
                v[i] = lo | (hi << 16);
            }
            ht[((size_t)(f >> 5) * n_groups + gr) * 32 + (f & 31)] = v;
        }
    }
}

struct SruWs {
    size_t u, h0, h1, wp, rws, prob, ht, total;
};

static SruWs sru_ws_layout(const sru_weights *w, int B, int L)
{
    SruWs s;
    size_t T = (size_t)B * L;
    if (T == 0) T = 1;
    int wide = w->n_in > w->n_hidden ? w->n_in : w->n_hidden;
    size_t off = 0;
    s.u = off;
    off += align_up(T * 4 * (size_t)w->n_hidden * sizeof(float), 256);
    s.h0 = off;
    off += align_up(T * (size_t)w->n_hidden * 2, 256);
    s.h1 = off;
    off += align_up(T * (size_t)w->n_hidden * 2, 256);
    s.wp = off;
    off += align_up((size_t)wide * 4 * w->n_hidden * 2, 256);
    s.rws = off;
    off += route_ws_bytes(w->n_hidden, w->n_out, MOE_BF16);
    s.prob = off;
    off += align_up(T * sizeof(float), 256);
    s.ht = off;
    if (w->attention) off += sru_attention_ws_bytes(B, L, w->n_hidden);
    s.total = off;
    return s;
}

static int sru_check(const sru_weights *w, int B, int L, int dtype)
{
    MOE_REQUIRE(w, MOE_ERR_INVALID_ARG, "sru_predict: null weights");
    MOE_REQUIRE(B >= 0 && L > 0 && w->n_layers > 0 && w->n_in > 0 && w->n_hidden > 0 && w->n_out > 0,
                MOE_ERR_INVALID_ARG, "sru_predict: B=%d L=%d layers=%d n_in=%d n_hidden=%d n_out=%d out of range", B, L,
                w->n_layers, w->n_in, w->n_hidden, w->n_out);
    MOE_REQUIRE((long long)B * L <= 0x7fffffffLL / 4096, MOE_ERR_UNSUPPORTED, "sru_predict: B*L too large");
    MOE_REQUIRE(dtype == MOE_BF16, MOE_ERR_UNSUPPORTED, "sru_predict: only MOE_BF16 is built");
    MOE_REQUIRE(w->n_in % 64 == 0 && w->n_hidden % 128 == 0, MOE_ERR_UNSUPPORTED,
                "sru_predict: n_in=%d must be a multiple of 64 and n_hidden=%d of 128", w->n_in, w->n_hidden);
    MOE_REQUIRE(w->n_out <= MOE_MAX_EXPERTS && w->n_out % 8 == 0, MOE_ERR_UNSUPPORTED,
                "sru_predict: n_out=%d must be a multiple of 8 and at most %d", w->n_out, MOE_MAX_EXPERTS);
    MOE_REQUIRE(B <= 65535, MOE_ERR_UNSUPPORTED, "sru_predict: B=%d exceeds 65535", B);
    MOE_REQUIRE(w->w_layout == MOE_LAYOUT_PLAIN || w->w_layout == MOE_LAYOUT_PACKED, MOE_ERR_INVALID_ARG,
                "sru_predict: unknown weight layout %d", w->w_layout);
    MOE_REQUIRE(w->attention == 0 || w->attention == 1, MOE_ERR_INVALID_ARG, "sru_predict: attention must be 0 or 1");
    MOE_REQUIRE(!w->attention || (L <= 1024 && w->n_hidden <= 256), MOE_ERR_UNSUPPORTED,
                "sru_predict: sparsemax attention needs L <= 1024 and n_hidden <= 256 (L=%d n_hidden=%d)", L,
                w->n_hidden);
    MOE_REQUIRE(w->w_layout == MOE_LAYOUT_PLAIN ||
                    ((w->n_out == 128 || w->n_out == 256) && w->n_hidden % 128 == 0),
                MOE_ERR_UNSUPPORTED, "sru_predict: packed weights need n_out = 128 or 256");
    return MOE_OK;
}

}  // namespace moe

using namespace moe;

extern "C" size_t sru_predict_workspace_bytes(const sru_weights *w, int B, int L, int dtype)
{
    if (sru_check(w, B, L, dtype) != MOE_OK) return 0;
    return sru_ws_layout(w, B, L).total;
}

extern "C" int sru_predict(const void *emb, const sru_weights *w, int B, int L, int dtype, int32_t *pred_idx,
                           float *logits_opt, void *ws, size_t ws_bytes, void *stream)
{
    int rc = sru_check(w, B, L, dtype);
    if (rc != MOE_OK) return rc;
    MOE_REQUIRE(w->w_cat && w->w_head, MOE_ERR_INVALID_ARG, "sru_predict: null weight table");
    for (int l = 0; l < w->n_layers; ++l)
        MOE_REQUIRE(w->w_cat[l] && aligned16(w->w_cat[l]), MOE_ERR_INVALID_ARG,
                    "sru_predict: w_cat[%d] null or misaligned", l);
    if (B == 0) return MOE_OK;
    MOE_REQUIRE(emb && pred_idx && aligned16(emb), MOE_ERR_INVALID_ARG, "sru_predict: null or misaligned pointer");
    SruWs lay = sru_ws_layout(w, B, L);
    MOE_REQUIRE(ws && aligned16(ws) && ws_bytes >= lay.total, MOE_ERR_WORKSPACE,
                "sru_predict: workspace of %zu bytes needed, %zu given", lay.total, ws_bytes);
    hipStream_t st = (hipStream_t)stream;
    char *base = (char *)ws;
    float *U = (float *)(base + lay.u);
    bf16_t *hbuf[2] = {(bf16_t *)(base + lay.h0), (bf16_t *)(base + lay.h1)};
    void *wp = base + lay.wp;
    const int T = B * L, n_h = w->n_hidden;
    // a packed head is only usable by the matrix-core head kernel; otherwise the head stays plain
    const int head_layout = w->w_layout;
    const bf16_t *cur = (const bf16_t *)emb;
    int nin = w->n_in;
    bool packed = false;                       // cur is a fragment image
    bool packed_in_h = false;                  // which lies in the two state buffers
    // the attention reads fragments from a one-kernel layer, which also writes the image of its weighted sums
    const bool later_two = !w->attention && sru_two_kernels(B, L, n_h, n_h, true, false);
    const bool first_two = !(w->attention && w->n_layers == 1) &&
                           sru_two_kernels(B, L, nin, n_h, false, w->n_layers > 1 && !later_two);
    const bool dealt = sru_deals_channels(B, L, nin, n_h, w->n_layers, first_two, later_two);
    if (!first_two && fus_packs_input(B, L, nin, n_h)) {
        bf16_t *image = (bf16_t *)(base + lay.u + fus_image_bytes(B, L, n_h));
        const int units = ceil_div(L, 32) * (nin / 64) * B;
        hipLaunchKernelGGL(sru_pack_input_kernel, dim3((int)align_up((size_t)units, 8)), dim3(256), 0, st, (const uint4 *)cur, units, L, nin,
                           (uint4 *)image);
        MOE_CHECK_LAUNCH("sru_predict/pack_input");
        cur = image;
        packed = true;
    }
    for (int l = 0; l < w->n_layers; ++l) {
        int k = nin == n_h ? 3 : 4;
        int ncol = k * n_h;
        const void *wl = w->w_cat[l];
        if (w->w_layout == MOE_LAYOUT_PLAIN) {
            rc = pack_matrix_launch(w->w_cat[l], nin, ncol, wp, st, "sru_predict/pack");
            if (rc != MOE_OK) return rc;
            wl = wp;
        }
        // Every one-kernel layer but the last hands its states on as a fragment image (the last does so to the attention), if they are
        // read by such a layer; so does the scan of the first layer.  The images live in the room that the two-kernel form has for
        // its projections, which holds two of them from 8 positions on (blocks of 32 positions, padded).  The scan's lies in the two
        // state buffers, since it reads the projections as it writes; the layer after it then has its states where the images go.
        const bool last = l + 1 == w->n_layers, two = l == 0 ? first_two : later_two;
        const bool pin = packed;
        const bool pout = L <= FUS_MAX_L && L >= 8 &&
                          (last ? w->attention && sru_attention_takes_fragments(L) : !later_two);
        bf16_t *const image = (bf16_t *)(base + lay.u + (l & 1) * fus_image_bytes(B, L, n_h));
        bf16_t *const out = two ? hbuf[pout ? 0 : l & 1] : pout || packed_in_h ? image : hbuf[l & 1];
        packed = pout;
        packed_in_h = two && pout;
        if (!two) {
            // weights through LDS where they fit beside what else is there (K / 16 fragments of 1 KB; the row-major kernel of short
            // sequences keeps its LDS small, two to four of its workgroups share a CU).  For fragments of 257 .. 768 channels at 257 .. 512 positions that
            // is 10 % of a predictor on average over 40 of them (2 .. 4 layers, 384 .. 768 channels), us with every wavefront loading them and so:
            // 2 x 401, 384 channels, two layers 21.1, 20.2; 29 x 408, 640 channels, four 425, 367; 2 x 512, 768 channels, four 62.1, 55.1.
#define MOE_FUS_BUILD(N, PIN, WF) (dealt ? sru_layer_fused_kernel<N, PIN, WF, true> : sru_layer_fused_kernel<N, PIN, WF, false>)
#define MOE_FUS(N)                                                                                    \
    (pin ? (nin <= 256            ? MOE_FUS_BUILD(N, true, 2)                                         \
            : N > 1 && nin <= 768 ? MOE_FUS_BUILD(N, true, (N > 1 ? 6 : 2))                           \
                                  : MOE_FUS_BUILD(N, true, 0))                                        \
         : (N > 1 && nin <= 256   ? MOE_FUS_BUILD(N, false, (N > 1 ? 2 : 0))                          \
            : N > 1 && nin <= 768 ? MOE_FUS_BUILD(N, false, (N > 1 ? 6 : 0))                          \
                                  : MOE_FUS_BUILD(N, false, 0)))
            auto fused = L <= 256 ? MOE_FUS(1) : L <= 512 ? MOE_FUS(2) : MOE_FUS(4);
#undef MOE_FUS
#undef MOE_FUS_BUILD
            hipLaunchKernelGGL(fused, dim3((n_h / FUS_CH) * B), dim3(FUS_THREADS), 0, st, cur, (const bf16_t *)wl, L, nin, n_h, k,
                               w->b_f ? w->b_f[l] : nullptr, w->b_r ? w->b_r[l] : nullptr, pout ? 1 : 0, out,
                               last && pout ? (bf16_t *)(base + lay.ht) : nullptr);
            MOE_CHECK_LAUNCH("sru_predict/layer");
            cur = out;
            nin = n_h;
            continue;
        }
        hipLaunchKernelGGL(sru_proj_kernel, dim3(ceil_div(T, 64) * (ncol / 128)), dim3(GEMM_THREADS), 0, st, cur,
                           (const bf16_t *)wl, T, nin, ncol, U);
        MOE_CHECK_LAUNCH("sru_predict/proj");
        auto scan = L <= 16 * SRU_CHUNKS ? sru_scan_kernel<16> : sru_scan_kernel<0>;
        hipLaunchKernelGGL(scan, dim3(n_h / SRU_CHANNELS, B), dim3(SRU_CHUNKS * SRU_CHANNELS), 0, st, U, cur, L,
                           n_h, k,
                           w->b_f ? w->b_f[l] : nullptr, w->b_r ? w->b_r[l] : nullptr, pout ? 1 : 0, out);
        MOE_CHECK_LAUNCH("sru_predict/scan");
        cur = out;
        nin = n_h;
    }
    if (w->attention) {
        bf16_t *zbuf = hbuf[w->n_layers & 1];      // the buffer the last layer did not write
        rc = sru_attention_launch(cur, packed, B, L, n_h, zbuf, base + lay.ht, st, "sru_predict/attention");
        if (rc != MOE_OK) return rc;
        cur = zbuf;
    }
    return route_launch(cur, w->w_head, head_layout, w->b_head, T, n_h, w->n_out, MOE_BF16, 1, 0, pred_idx, (float *)(base + lay.prob),
                        logits_opt, base + lay.rws, st, "sru_predict/head");
}
