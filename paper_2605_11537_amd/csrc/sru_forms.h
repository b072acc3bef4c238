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
// with it: 16 x 1024, 768 -> 256: 112 and 95 us, 512 -> 256: 87 and 80; 8 x 1024, 768 -> 256: 57 and 50; 5 x 777: 44 and 42; at up to 512
// positions 1 .. 3 us more with it.
static inline bool fus_packs_input(int B, int L, int K, int n_h)
{
    return L > 512 && L <= FUS_MAX_L && K >= 512 &&
           fus_image_bytes(B, L, n_h) + fus_image_bytes(B, L, K) <= (size_t)B * L * 4 * n_h * sizeof(float);
}

// Projection and scan in two kernels, or the layer in one?  One kernel up to 512 positions, two above 1024.  Between them one
// workgroup fills a CU and reads all rows of its sequence, so its time grows with K, in steps of 256 workgroups (rounds, of which
// share is filled), while the two kernels deal the work out evenly but send the projections through memory (dearer from 10 million
// on, 40 MB).  The estimates (microseconds; K and L in thousands, x in millions of projections) were fitted to 300 layers of 1 .. 200
// sequences of 513 .. 1024 positions, 64 .. 2048 -> 128 .. 1024 channels, with a one-kernel form in which every wavefront had the same number of row
// blocks and every chunk 16 steps; the present one is faster where a sequence does not fill them.  So the estimate for one kernel is too high
// there: taking the form they choose costs 3.1 % on average against always knowing (150 predictors of one to three such layers, 86 single ones
// 3.0 %; 0.3 % with the kernel that was fitted), up to 46 % (170 x 630, 384 -> 768: two kernels 1216 us, one 831), where two are taken
// and one would do.  One layer and the head, two against one kernel: 1 x 1024, 1024 -> 256: 28 and 40 us; 5 x 777, 1024 -> 1024: 76 and 90; 64 x 600, 1024 ->
// 1024: 634 and 694; 8 x 1024, 256 -> 256: 34 and 24; 16 x 1024, 768 -> 256: 79 and 63; 64 x 1024, 384 -> 384: 302 and 267.
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

// Which XCDs the workgroups of the one-kernel layers go to.  Whole sequences per XCD (ranges of them) have an L2 fetch 1/8 of the rows and all weights, channel
// blocks dealt to the XCDs 1/8 of the weights and all rows; as long as the weights stay in an XCD's 4 MB L2 from one call to the next, they are no
// matter.  So the channel blocks are dealt where an XCD's share of the predictor's weights does not fit (beside 3.8 MB of them there is
// no room) and the weights it would fetch outweigh seven times the rows: those of a layer, once for every XCD that has a sequence, or, past
// what stays through a layer (3.2 MB), for every sequence.  Captured, head included, us, ranges of sequences and dealt: 14 x 18, 768 -> 512, four
// layers 43.7, 40.5; 9 x 23, 768 -> 256, ten 71.1, 68.2; 30 x 41, 768 -> 1024, four 196, 172; 38 x 255, 768 -> 1024, three 511, 481; 12 x 512,
// 256 -> 256, four 67.8, 76.0.  Where they outweigh the rows sixteen times, sooner: the rows that dealing fetches 8 times are next to nothing there, and
// from 2.8 MB on some of an XCD's weights are gone by the next call (9 x 16, 960 -> 512, one layer 18.6, 17.2; 3 x 19, 1024 -> 768, two 19.3, 18.3; one
// sequence has its channel blocks on all XCDs either way).  Over 460 predictors whose sequences are no multiple of 8, and 250 next to these lines, the
// choice is at most 1.7 % slower than always dealt and 2.1 % (1.3 % next to the lines) faster on average.  Where something else has run in between (caches flushed)
// ranges are 2 .. 4 % ahead with either kind.
// Multiples of 8 keep their sequences together at any size.
static inline bool sru_deals_channels(int B, int L, int n_in, int n_h, int n_layers, bool first_two, bool later_two)
{
    if (B % 8 == 0) return false;
    const double mb = 1 << 20, held = B < 8 ? B : 8;
    double all = 0, fetched = 0, rows = 0;
    auto layers = [&](int n, int K) {
        const double weights = (double)K * (K == n_h ? 3 : 4) * n_h * 2 / mb;
        all += n * weights;
        fetched += n * weights * (weights > 3.2 ? B : held);
        rows += n * ((double)B * L * K * 2 / mb);
    };
    if (!first_two) layers(1, n_in);
    if (!later_two) layers(n_layers - 1, n_h);
    const double share = all * held / 8;
    return (share > 3.8 && fetched > 7 * rows) || (B > 1 && share > 2.8 && fetched > 16 * rows);
}

}  // namespace moe
