// How a projection of the prompt pass is laid out: which tile a workgroup has and how many pieces along K.  Host code alone.  Not installed.
#pragma once
#include <math.h>
#include <stddef.h>

#include "ad_prompt.h"

namespace ad {

constexpr int kLongPiece = 128;       // k-steps above which a piece's sums count as long (see k_prompt_gemm's accumulators)
constexpr int kShortestPiece = 8;     // fewest k-steps of a piece

// A kind of tile: 4 * wr row tiles by bt token tiles.  About `step` us go by per k-step, `round` more per round of a workgroup per compute
// unit, `piece` us and 1 / rate per byte for a piece after the first.  pair: two workgroups share a compute unit, so that 1.5 rounds take 1.5 times one's
// time and not two.  halves: tiles that would fill less than half of a last round are dealt as two of half the rows, whose k-step takes half_step.
struct PromptTileKind { int wr, bt; double step, half_step, round, piece, rate; bool pair, halves; };

// The fewest pieces along K: pieces of more than kLongPiece k-steps have long sums, and are taken only where more of them would leave the
// chip no room for other work (8B shape, 512 tokens, 14336 inputs: two pieces off by 1.08 times as much as four).
inline int fewest_pieces(const PromptGemm &g, int n_wg) {
    const int tiles = (g.NT + 7) / 8 * ((g.M + 127) / 128);
    int n = 1;
    while (n < kPromptMaxSplit && n * kLongPiece < g.KT && tiles * (n + 1) <= 2 * n_wg && (size_t)(n + 1) * g.M * g.N <= g.part_floats) ++n;
    return n;
}

// Lays the product out in such tiles and, with `pieces`, in the number of pieces along K that takes the least time; returns about how many microseconds.
inline double lay_out(PromptGemm &g, const PromptTileKind &t, bool pieces, int n_wg) {
    g.n_rb = (g.NT + 4 * t.wr - 1) / (4 * t.wr);
    g.n_tb = ((g.M + 15) / 16 + t.bt - 1) / t.bt;
    PromptGemm best = g;
    double least = INFINITY;
    const int fewest = pieces ? fewest_pieces(g, n_wg) : 1;
    for (int split = fewest; split <= (pieces ? kPromptMaxSplit : 1); ++split) {
        if (split > fewest && (g.KT / split < kShortestPiece || (size_t)split * g.M * g.N > g.part_floats)) break;
        PromptGemm h = g;
        h.k_per = (g.KT + split - 1) / split;
        h.n_split = (g.KT + h.k_per - 1) / h.k_per;
        const int tiles = h.n_rb * h.n_tb * h.n_split, rest = tiles % n_wg;
        const bool halves = t.halves && rest && 2 * rest <= n_wg;
        h.n_full = halves ? tiles - rest : tiles;
        const double round = t.round + h.k_per * t.step;
        double us = (double)(h.n_split - 1) * ((double)g.M * g.N * 4 / t.rate + t.piece);
        if (t.pair) us += round * (tiles <= n_wg ? 1.0 : (double)tiles / n_wg);
        else us += round * (tiles / n_wg) + (!rest ? 0.0 : halves ? t.round + h.k_per * t.half_step : round);
        if (us < least) {
            least = us;
            best = h;
        }
    }
    g = best;
    return least;
}

// Lays the product out in the tiles whose time is least; returns their kind.  Up to 64 tokens bound by the weights' way from memory, or, where a product has less than the chip's
// workgroups, by the chain through a workgroup's k-steps: 64 or 128 rows by 32 tokens, 128 by 64.  More: 8 wavefronts, 128, 192 or
// 256 rows by 96 or 128 tokens, so that the least of the last round and of the last token block is empty.  The times are fitted to the products of the
// 8B and 13B shapes and of models of 1024 and 2048 inputs at 16 to 1023 tokens, where the rule's choice takes 1.5 % (up to 64 tokens) and 2.6 %
// longer in the mean than the best of all tiles and pieces.
//
// Large products are bound by the matrix cores and, with them, by the power that operands on the move take: a loop of 16x16x32 products on registers alone reaches
// 1.92 PFLOP/s here with random operands (2.38 with zeros; 32x32x16 ones 1.78, their accumulators move twice as often), with operands from
// LDS as 4 x 4 tiles need them 1.75.  Larger wavefront tiles take fewer reads of LDS per product (12 for 32 with 4 x 4, 10 for 16 with 2 x 4).  One
// wavefront per SIMD with 8 x 4 tiles, and 32x32x16 products, were slower.  Measured with weights that no cache holds, us for 6144 x 4096, 4096 x
// 4096, 4096 x 14336, 28672 x 4096, against 2 x 4 tiles for every product, all operands read at the start of a step, power-of-two pieces:
//     16 tokens   11.8    8.3   21.8   43.2     13.8    9.9   23.8   45.9
//     64          15.5   11.9   27.2   47.3     20.5   14.0   29.6   53.3
//    160          26.4   20.8   48.3   76.9     36.3   29.4   62.7  127
//    256          32.8   24.0   57    102       39.7   33.0   66.5  127
//    640          56.6   43.1  138    301       66.5   58.8  207    337
//   1023          84     59    173    368      113     68    205    412    (within a prompt of 8 layers; 1.16 to 1.39 PFLOP/s, hi and lo products both counted)
constexpr int kPromptTileKinds = 9;
inline int choose_prompt_tile(PromptGemm &g, bool pieces, int n_wg) {
    auto step8 = [](int n) { return 0.093 + 0.0356 * n; };      // 8 wavefronts of n accumulators
    auto large = [&](int wr, int wt) { return PromptTileKind{wr, 2 * wt, step8(wr * wt), step8(wr * wt / 2), 2, 0.5, 1.5e6, false, wr == 4}; };
    const PromptTileKind kinds[kPromptTileKinds] = {
        {1, 2, 0.12, 0, 0, 0.1, 2e6, true, false}, {2, 2, 0.19, 0, 0, 0.1, 2e6, false, false}, {2, 4, 0.24, 0, 0, 0.1, 2e6, false, false},
        large(2, 3), large(2, 4), large(3, 3), large(3, 4), large(4, 3), large(4, 4)};
    const PromptGemm plain = g;
    double least = INFINITY;
    int kind = 0;
    for (int i = g.M <= 64 ? 0 : 3; i < (g.M <= 64 ? 3 : 9); ++i) {
        PromptGemm h = plain;
        const double us = lay_out(h, kinds[i], pieces, n_wg);
        if (us < least) {
            least = us;
            g = h;
            kind = i;
        }
    }
    return kind;
}

}  // namespace ad
