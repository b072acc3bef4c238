// bf16 grouped product for batches between the two others: more rows per expert than the weight-streaming kernel is made for (64 on
// average), but not enough of them to give every CU a 256 x 256 tile.
//
// 128 rows of one expert x 64 * NB columns per workgroup (128 or 256), two workgroups per CU.  Both operands go global -> LDS directly
// into a ring of 32-k stages, as in the 256 x 256 kernel; the four wavefronts are a 2 x 2 grid of 64 x 32 NB outputs.  The fragments of the
// next 16-deep step are read while the current ones are multiplied, one barrier per stage.  The loads of a stage are spread over the matrix
// instructions as there, where a wavefront has two row blocks (all behind the barrier and so, both products, us: 768 x 3072, 16 experts x 627 rows
// 118, 113, 8 x 1024 103, 95; 384 x 1536, 32 x 349 57, 54; no change where tiles are few).  A workgroup finds its tile in the slot tables
// (ffn_share.h), so there is no list kernel in front.
//
// Bound: what a CU gets from beyond its L2, about 50 GB/s, as first readers of weights and of h (8 experts x 90 rows, k = 4096, 64
// workgroups of 1.8 MB each: 36 us), and with two workgroups per CU the load path and LDS together.  More stages in flight (six of 24 KB, nine of 16 KB, one
// workgroup per CU) and stages of 64 k left the times where they are or lost 10 .. 30 %.
// Measured, both products with what is launched in front of them, us: 256 x 256 kernel (128-column kernel where that does not apply), this one:
//   512 x 2048, 16 experts x 480 rows: 69, 51      768 x 3072, 16 x 627: 132, 112      1024 x 4096, 8 x 393: 136, 78
//   256 x 1024, 16 x 512: 41, 26                   384 x 1536, 32 x 349: 62, 54        1024 x 4096, 8 x 90: 57, 49
#pragma once
#include "ffn_share.h"
#include "gemm_dense_bf16.h"

namespace moe {

constexpr int MID_BM = 128, MID_BK = 32;

template <int NB>
struct MidTile {
    static constexpr int BN = 64 * NB;
    static constexpr int NS = NB == 2 ? 4 : 3;                   // stages in the ring: 64 or 72 KB
    static constexpr int A_UNITS = MID_BM / 16, B_UNITS = 4 * NB; // 1 KB each, what a wavefront-wide load brings
    static constexpr int STAGE = (A_UNITS + B_UNITS) * 64;       // 16-byte pieces
    static constexpr int LDE = 32 * NB + 8;                      // epilogue strip row stride, elements
};

template <bool RELU, int NB>
__global__ __launch_bounds__(SHARE_THREADS, 2) void ffn_lds_tile_bf16_kernel(
    const bf16_t *__restrict__ A, const bf16_t *__restrict__ Wp, const int32_t *__restrict__ row_index, int n_src_rows, int K,
    int N, int E, const int32_t *__restrict__ slot_offset, const int32_t *__restrict__ slot_expert,
    const int32_t *__restrict__ n_slots_p, int max_slots, int max_rows, bf16_t *__restrict__ C)
{
    using Tile = MidTile<NB>;
    constexpr int NS = Tile::NS, STAGE = Tile::STAGE, LDE = Tile::LDE, BN = Tile::BN, BK = MID_BK;
    constexpr int AU = 2, BU = NB;                               // units a wavefront loads per stage
    static_assert(NS * STAGE * 16 >= 4 * 32 * LDE * 2, "the epilogue strips lie in the ring");
    __shared__ __attribute__((aligned(16))) uint4 ring[NS * STAGE];
    __shared__ TileItem found;
    TileShare<MID_BM> share;
    share.E = E;
    share.schedule = MOE_SCHEDULE_SLOTS;
    share.n_nt = N / BN;
    share.max_rows = max_rows;
    share.find(slot_offset, slot_expert, n_slots_p, max_slots, &found);
    const int unit = share.first + (int)(blockIdx.x >> 3);
    if (unit >= share.end) return;                               // uniform
    share.write_item(slot_offset, slot_expert, unit, &found);
    __syncthreads();
    const TileItem it = found;
    if (it.expert < 0 || it.expert >= E || it.row_begin < 0) return;         // uniform; never index with a bad table
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), wm = w >> 1, wn = w & 1;
    const int row_end = it.row_end < max_rows ? it.row_end : max_rows;
    const int nk = K / BK, KG = K >> 3;
    const unsigned lds0 = (unsigned)(unsigned long)(lds_void_t *)ring;
    // A token unit is 16 rows x 4 k-groups; row r's group g lies at piece 4 r + (g ^ (r >> 2) ^ (r & 3)), so that the lanes of a fragment
    // read fall on different banks.  A weight unit is a strip's fragment of 16 k as the packed image has it.
    const int r16 = lane & 15;
    unsigned a_addr[2];                                          // of this lane's pieces of row block wm in stage 0
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int kg = 2 * ks + (lane >> 5);
        a_addr[ks] = lds0 + 16u * ((wm * 2 + ((lane & 31) >> 4)) * 64 + r16 * 4 + (kg ^ (r16 >> 2) ^ (r16 & 3)));
    }
    const unsigned b_addr = lds0 + 16u * ((Tile::A_UNITS + wn * NB * 2) * 64 + lane);
    const int ld_r = lane >> 2, ld_kg = (lane & 3) ^ (ld_r >> 2) ^ (ld_r & 3);
    const uint4 *b_src[BU];
#pragma unroll
    for (int i = 0; i < BU; ++i) {
        const int u = w * BU + i;
        b_src[i] = reinterpret_cast<const uint4 *>(Wp + (size_t)it.expert * K * N) +
                   ((size_t)(it.column * 2 * NB + (u >> 1)) * KG + (u & 1) * 2) * 32 + lane;
    }
    const int r0 = it.row_begin, nrows = row_end - r0;           // 1 .. 128: a tile has a row
    if (nrows <= 0) return;
    const int blocks = (nrows + 31) >> 5;
    const bool own_rows = w < blocks;                        // this wavefront loads block w of the rows
    int src[AU];
#pragma unroll
    for (int i = 0; i < AU; ++i) {
        const int r = 32 * w + 16 * i + ld_r;
        src[i] = r0 + (r < nrows ? r : nrows - 1);           // rows past the tile repeat its last row
    }
    if (row_index) {
#pragma unroll
        for (int i = 0; i < AU; ++i) src[i] = row_index[src[i]];
#pragma unroll
        for (int i = 0; i < AU; ++i) src[i] = src[i] >= 0 && src[i] < n_src_rows ? src[i] : 0;       // a bad index reads row 0
    }
    const bf16_t *a_src[AU];
#pragma unroll
    for (int i = 0; i < AU; ++i) a_src[i] = A + (size_t)src[i] * K + ld_kg * 8;
    MOE_VMCNT(0);                                            // from here on only the stages' loads are counted
    // stage kc's loads, tokens and weights apart; past the end: a harmless re-read
    auto load_a = [&](int kc, int buf, int i) {
        const int k = kc < nk ? kc : nk - 1;
        __builtin_amdgcn_global_load_lds((glb_void_t *)(a_src[i] + k * BK), (lds_void_t *)(ring + buf * STAGE + (AU * w + i) * 64), 16, 0, 0);
    };
    auto load_b = [&](int kc, int buf, int i) {
        const int k = kc < nk ? kc : nk - 1;
        __builtin_amdgcn_global_load_lds((glb_void_t *)(b_src[i] + (size_t)k * (BK / 8) * 32),
                                         (lds_void_t *)(ring + buf * STAGE + (Tile::A_UNITS + w * BU + i) * 64), 16, 0, 0);
    };
    // all but the newest `young` stages have landed -- of them `late` loads are still to be asked for --, for everybody behind the barrier
    auto landed = [&](auto YOUNG, auto LATE) {
        constexpr int young = decltype(YOUNG)::value, late = decltype(LATE)::value;
        if (own_rows) MOE_VMCNT(young * (BU + AU) - late);
        else MOE_VMCNT(young * BU - late);
        __builtin_amdgcn_s_barrier();
        MOE_SB();
    };
    // one body per number of row blocks (2 * mb + wm) a wavefront owns
    auto run_tile = [&](auto BLOCKS) {
        constexpr int MYB = decltype(BLOCKS)::value;
        // SPREAD: the loads of a stage between the matrix instructions, its weights half a stage after its tokens.  A wavefront with one row block or
        // none has half the instructions to hide them behind and waits for them: all at once behind the barrier (both products, us, spread and so: 70 rows
        // of which 56 are kept, 1024 x 4096 41.8, 38.0; 8 x 56, 1024 x 2048 29.8, 27.4; 6 x 44, 512 x 2048 26.0, 23.8).  Every wavefront waits for its
        // own loads, so both kinds share the ring.
        constexpr bool SPREAD = MYB > 1;
        f32x16_t acc[MYB ? MYB : 1][NB];
        zero_acc<MYB ? MYB : 1, NB>(acc);
        u32x4_t fx[2 + NB], fy[2 + NB];                          // fragments of two 16-deep steps: two row blocks, NB strips
        auto read = [&](u32x4_t (&f)[2 + NB], int ks, int buf) {
            const unsigned a = a_addr[ks] + buf * (STAGE * 16), b = b_addr + buf * (STAGE * 16) + ks * 1024;
            if constexpr (MYB == 0) f[0] = (u32x4_t){0u, 0u, 0u, 0u};
            else MOE_DS_READ128(f[0], a, 0);
            if constexpr (MYB < 2) f[1] = (u32x4_t){0u, 0u, 0u, 0u};
            else MOE_DS_READ128(f[1], a, 4096);
            MOE_DS_READ128(f[2], b, 0);
            MOE_DS_READ128(f[3], b, 2048);
            if constexpr (NB == 4) {
                MOE_DS_READ128(f[4], b, 4096);
                MOE_DS_READ128(f[5], b, 6144);
            }
            MOE_SB();
        };
        // the registers are operands so that no use of them can move above the wait
        auto wait = [&](u32x4_t (&f)[2 + NB]) {
            if constexpr (NB == 4)
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]), "+v"(f[5]));
            else
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]));
            MOE_SB();
        };
        // (weights, tokens): the transposed block, a lane holds 4 consecutive columns of one token
        // between(i) follows matrix instruction i where the loads are spread
        auto multiply = [&](const u32x4_t (&f)[2 + NB], auto between) {
#pragma unroll
            for (int mb = 0; mb < MYB; ++mb)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, f[2 + nb]),
                                                                          __builtin_bit_cast(bf16x8_t, f[mb]), acc[mb][nb], 0, 0, 0);
                    if constexpr (SPREAD) {
                        between(mb * NB + nb);
                        MOE_SB();
                    }
                }
            MOE_SB();
        };
        using std::integral_constant;
        auto load_stage = [&](int kc, int buf, auto WEIGHTS) {
            if (own_rows) {
#pragma unroll
                for (int i = 0; i < AU; ++i) load_a(kc, buf, i);
            }
            if constexpr (decltype(WEIGHTS)::value) {
#pragma unroll
                for (int i = 0; i < BU; ++i) load_b(kc, buf, i);
            }
            MOE_SB();
        };
#pragma unroll
        for (int s = 0; s + 1 < NS; ++s) load_stage(s, s, std::true_type{});
        load_stage(NS - 1, NS - 1, integral_constant<bool, !SPREAD>{});
        landed(integral_constant<int, NS - 1>{}, integral_constant<int, SPREAD ? BU : 0>{});
        int buf = 0, late_buf = NS - 1;
        read(fx, 0, 0);
        wait(fx);
        for (int kc = 0; kc < nk; ++kc) {
            read(fy, 1, buf);
            multiply(fx, [&](int i) {                        // a load per two of them: the weights of the stage whose tokens went out last
                if (i % 2 == 0 && i / 2 < BU) load_b(kc + NS - 1, late_buf, i / 2);
            });
            wait(fy);
            // behind the barrier stage kc + 1 is there and stage kc has been read by all
            landed(integral_constant<int, NS - 2>{}, integral_constant<int, 0>{});
            if constexpr (!SPREAD) load_stage(kc + NS, buf, std::true_type{});
            late_buf = buf;
            buf = buf + 1 == NS ? 0 : buf + 1;
            read(fx, 0, buf);
            multiply(fy, [&](int i) {
                if (own_rows && i % 2 == 0 && i / 2 < AU) load_a(kc + NS, late_buf, i / 2);
            });
            wait(fx);
        }
        MOE_VMCNT(0);                                            // the re-reads past the end
        barrier_anywhere();                                      // everybody has read the last stage: the strips take its place
        bf16_t *strip = reinterpret_cast<bf16_t *>(ring) + w * (32 * LDE);
#pragma unroll
        for (int mb = 0; mb < MYB; ++mb) {
            const int first = (2 * mb + wm) * 32;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = RELU ? fmaxf(acc[mb][nb][4 * q + i], 0.f) : acc[mb][nb][4 * q + i];
                    *reinterpret_cast<uint2 *>(strip + (lane & 31) * LDE + nb * 32 + 8 * q + 4 * (lane >> 5)) =
                        make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            constexpr int PPR = 4 * NB, RPI = 64 / PPR;          // 16-byte pieces per row, rows per instruction
#pragma unroll
            for (int i = 0; i < 32 / RPI; ++i) {
                const int r = i * RPI + lane / PPR;
                if (first + r < nrows)
                    *reinterpret_cast<uint4 *>(C + (size_t)(r0 + first + r) * N + it.column * BN + wn * 32 * NB + (lane % PPR) * 8) =
                        *reinterpret_cast<const uint4 *>(strip + r * LDE + (lane % PPR) * 8);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    };
    const int my_blocks = (blocks - wm + 1) >> 1;
    using std::integral_constant;
    // (the short bodies first: behind the long one their instructions arrive later, 1 .. 2 % of tiles of up to 64 rows)
    if (my_blocks == 1) run_tile(integral_constant<int, 1>{});
    else if (my_blocks == 0) run_tile(integral_constant<int, 0>{});
    else run_tile(integral_constant<int, 2>{});
}

// Columns per workgroup in units of 64: 256 where those tiles fill the chip, else 128 (1024 x 4096, 8 experts x 90 rows: first product 20.9
// against 15.7 us; 512 x 2048, 16 x 480 rows: 27 against 34).
static inline int mid_strips(int max_rows, int max_slots, int N)
{
    const long long tiles = max_rows / MID_BM + max_slots / 2;
    return N % 256 == 0 && tiles * (N / 256) >= 256 ? 4 : 2;
}

}  // namespace moe
