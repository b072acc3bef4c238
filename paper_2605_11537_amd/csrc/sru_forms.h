// Which kernels an SRU layer runs on: host rules.
#pragma once
#include "common.h"

namespace moe {

constexpr int FUS_CH = 8;              // channels per workgroup of the one-kernel layer
constexpr int FUS_MAX_L = 1024;        // positions it holds

// bytes of the fragment image of B sequences of L states of n channels (at most half of B*L*4*n binary32 values if L >= 8)
static inline size_t fus_image_bytes(int B, int L, int n) { return (size_t)B * align_up((size_t)L, 32) * n * 2; }

// The longest sequences of wide embeddings have them packed once, where the row-major kernel turns them into fragments in each
// of the n_hidden / 8 workgroups of a sequence.  The image lies where the second layer's states go afterwards, behind the first's,
// if the room for the projections holds it.  Measured where the one-kernel form is taken, two layers and the head without and
// with it: 16 x 1024, 768 -> 256: 109 and 91 us, 512 -> 256: 86 and 80; 8 x 1024, 768 -> 256: 59 and 53; at up to 512
// positions 2 .. 7 us more with it.
static inline bool fus_packs_input(int B, int L, int K, int n_h)
{
    return L > 512 && L <= FUS_MAX_L && K >= 512 &&
           fus_image_bytes(B, L, n_h) + fus_image_bytes(B, L, K) <= (size_t)B * L * 4 * n_h * sizeof(float);
}

// Projection and scan in two kernels, or the layer in one?  One kernel up to 512 positions, two above 1024.  Between them one
// workgroup fills a CU and reads all rows of its sequence, so its time grows with K, in steps of 256 workgroups (rounds, of which
// share is filled), while the two kernels deal the work out evenly but send the projections through memory (dearer from 10 million
// on, 40 MB).  The estimates (microseconds; K and L in thousands, x in millions of projections) are fitted to 300 layers of 1 .. 200
// sequences of 513 .. 1024 positions, 64 .. 2048 -> 128 .. 1024 channels, with mean errors of at most 12 and 8 %; taking the form they
// choose costs 0.3 % on average against always knowing.  Two against one kernel: 1 x 1024, 1024 -> 256: 25 and 35 us;
// 5 x 777, 1024 -> 1024: 68 and 94; 64 x 600, 1024 -> 1024: 640 and 972; 8 x 1024, 256 -> 256: 29 and 15; 16 x 1024, 768 -> 256:
// 73 and 60; 64 x 1024, 384 -> 384: 303 and 269.
// from_fragments: the one-kernel form would read its states as the layer before leaves them.  hands_on: the next layer is one kernel; the
// scan's states reach it 0.5 us (1 x 1024, 128 channels) to 3.5 us (5 x 777, 256 channels) later than those of a kernel of its own kind.
static inline bool sru_two_kernels(int B, int L, int K, int n_h, bool from_fragments, bool hands_on)
{
    if (L <= 512) return false;
    if (L > FUS_MAX_L) return true;
    const double k = K / 1e3, l = L / 1e3, x = (double)B * L * n_h * (K == n_h ? 3 : 4) / 1e6;
    const double two = 10.5 + 7.7 * l + 1.5 * k * l + (1.37 + 1.74 * k) * x + (x > 10 ? (2.2 - 0.9 * k) * (x - 10) : 0) +
                       (!hands_on ? 0 : x < 3 ? 0.5 + 0.8 * x : 3);
    const bool packs = !from_fragments && fus_packs_input(B, L, K, n_h);
    const double wgs = (double)B * (n_h / FUS_CH);
    const int rounds = (int)((wgs + 255) / 256);
    const double share = wgs / (256.0 * rounds);
    const double row = from_fragments || packs ? 10.4 * k + 10.3 * k * l : 15 * k + (13.9 + 8.4 * share) * k * l;
    const double one = rounds * (6.4 + 2.6 * share + row) + (packs ? 5 + 0.55 * B * l * k : 0);
    return two < one;
}

}  // namespace moe
