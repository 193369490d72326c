// Tiles of the K-slices form of the 16-bit products (gemm_bf16_slices.hpp) and the rule that takes it.
#pragma once
#include <stdint.h>

#include "ks_common.hpp"

namespace ks {

// KS_SLICES(index, BM, BN, BK, waves, stages, FIXED): FIXED us of a call around the K loop
#define KS_SLICES_TILES(X)             \
    X(0, 16, 16, 64, 8, 4, 2.79)       \
    X(1, 32, 16, 64, 8, 3, 2.71)       \
    X(2, 16, 32, 64, 8, 3, 2.65)       \
    X(3, 32, 32, 64, 8, 2, 2.75)       \
    X(4, 64, 16, 64, 4, 3, 2.81)       \
    X(5, 16, 64, 64, 4, 3, 2.82)       \
    X(6, 64, 32, 64, 4, 3, 3.64)       \
    X(7, 32, 64, 64, 4, 3, 3.53)       \
    X(8, 64, 64, 32, 8, 2, 3.49)       \
    X(9, 64, 64, 64, 4, 2, 6.59)
// and of the form for any operands: K-steps in registers in place of the stages
#define KS_SLICES_STAGED_TILES(X)      \
    X(10, 16, 16, 64, 16, 4, 2.80)     \
    X(11, 32, 16, 64, 8, 3, 2.93)      \
    X(12, 16, 32, 64, 8, 3, 2.90)      \
    X(13, 32, 32, 64, 8, 3, 3.12)      \
    X(14, 64, 16, 64, 8, 3, 3.52)      \
    X(15, 16, 64, 64, 8, 3, 3.36)      \
    X(16, 64, 32, 64, 8, 2, 3.84)      \
    X(17, 32, 64, 64, 8, 2, 3.76)      \
    X(18, 64, 64, 32, 8, 3, 4.49)
struct SliceTile {
    int bm, bn, bk, waves, stages;
    double fixed;
};
constexpr SliceTile kSliceTiles[] = {
#define KS_ROW(i, BM, BN, BK, NW, ST, FIXED) {BM, BN, BK, NW, ST, FIXED},
    KS_SLICES_TILES(KS_ROW) KS_SLICES_STAGED_TILES(KS_ROW)
#undef KS_ROW
};
constexpr int kSliceTilesAligned = 10;

// variant: 1 bkc, 2 akc, 16 binary16; stream: which operands are loaded past the last-level cache
void launch_bf16_slices(int tile, const GemmParams &p, int grid, int variant, int stream, hipStream_t s);

// Members that the form may stand in for, and sizes that may be one round of its largest tiles.
inline int slices_member(int id) { return id == 13 ? 0 : id == 27 ? 1 : id == 38 ? 2 : id == 39 ? 3 : -1; }
inline bool slices_possible(int id, int64_t M, int64_t N, int64_t K) {
    return slices_member(id) >= 0 && K >= 256 && ((M + 63) / 64) * ((N + 63) / 64) <= 256;
}
// K from 512 (any operands: 256) on, below which it is level.  Any operands: rows of seven elements at least; none of 64 MiB and more
// (up to 1.39 of the time), nor 1e10 flop, where copies pay.
inline bool slices_worth(bool staged, bool akc, bool bkc, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb) {
    if (!staged) return K >= 512;
    return (akc || lda >= 7) && (bkc || ldb >= 7) && M * K < (32LL << 20) && N * K < (32LL << 20) && 2.0 * (double)M * (double)N * (double)K < 1e10;
}

// us per 1024 of K that a compute unit's memory pipe takes for one operand of a tile of `extent` rows (of columns): a K-contiguous
// one by its bytes, of a row-contiguous one with less than 64 every k takes as long as a whole line; K-steps of 32 have
// K-contiguous pieces of 64 bytes.  staged: the form for any operands.
constexpr double slice_operand_us(bool staged, int extent, bool kc, int bk) {
    if (staged) {
        if (bk == 32) return kc ? 3.12 : 2.77;
        return extent == 16 ? (kc ? 0.58 : 1.35) : extent == 32 ? (kc ? 1.15 : 1.64) : (kc ? 2.29 : 2.40);
    }
    if (bk == 32) return kc ? 2.09 : 2.03;
    return extent == 16 ? (kc ? 0.34 : 1.12) : extent == 32 ? (kc ? 0.66 : 1.33) : (kc ? 1.23 : 1.61);
}
// Estimate for one round of work-groups of tile `t`, us: the longest of a unit's memory pipe, memory (a row-contiguous operand in
// pieces of less than a line is fetched as often as a line has pieces), what a work-group has in flight of an operand that comes
// from memory behind its 2 us (one of 64 MiB and more: 2944 x 2 x 14976 NT 18.4 us by the member, 22.7 in 184 tiles of 16 x 16) or from
// the last-level cache behind 0.8 (32 MiB: 2944 x 52 x 8960 NT 14.7 and 15.8), and the L2s.  Where the rows of an aligned K-contiguous
// operand do not begin at lines of 128 bytes, the piece of a K-step lies in one line more, which shows in tiles of 32 of its
// rows and more (1984 x 448 x 3584 NT, rows of 3592, 20.2 and 24.5).  The constants are fitted to the times of all tiles over 1300 (any
// operands: 1597) drawn products, 14 % (17 %) rms.
// (The tile is a template argument: a small call waits for the host, and with the constants folded ten estimates take it
// 10 to 60 ns where a loop over the table takes 45 to 100.)
struct SliceCall {
    bool akc, bkc;
    int64_t M, N;
    double k, latency;               // latency: us of a wave's round trip x K, 0 where all operands come from the L2s
    double aLines, bLines;           // what rows that do not begin at lines add to an operand's part
};
template <int T>
inline bool slices_us(const SliceCall &c, double &us) {
    constexpr SliceTile t = kSliceTiles[T];
    constexpr bool staged = T >= kSliceTilesAligned;
    const int64_t tiles = ((c.M + t.bm - 1) / t.bm) * ((c.N + t.bn - 1) / t.bn);
    if (tiles > 256) return false;
    constexpr double aKc = slice_operand_us(staged, t.bm, true, t.bk), aRc = slice_operand_us(staged, t.bm, false, t.bk),
                     bKc = slice_operand_us(staged, t.bn, true, t.bk), bRc = slice_operand_us(staged, t.bn, false, t.bk);
    double longest = c.k * (1.0 / 1024) * ((c.akc ? (t.bm >= 32 ? aKc * c.aLines : aKc) : aRc) +
                                           (c.bkc ? (t.bn >= 32 ? bKc * c.bLines : bKc) : bRc));
    const double memory = c.k * (2e-6 / (staged ? 6.14 : 5.99)) * ((double)c.M * (c.akc ? 1 : 64 / t.bm) + (double)c.N * (c.bkc ? 1 : 64 / t.bn));
    if (memory > longest) longest = memory;
    const double l2 = (double)tiles * c.k * ((t.bm + t.bn) * 2e-6 / (staged ? 10.66 : 17.02));
    if (l2 > longest) longest = l2;
    const double latency = c.latency * (1.0 / (t.waves * (t.stages - 1) * t.bk));
    if (latency > longest) longest = latency;
    const double x = t.fixed + longest;
    if (x >= us) return false;
    us = x;
    return true;
}
// The same for the member (id) that the call would run otherwise, `steps` K-steps in each of `groups` work-groups;
// partitions > 1: their sums are `partialBytes` and a second launch adds them.
inline double slices_other_us(bool staged, int id, int64_t M, int64_t N, int64_t K, int64_t groups, int64_t steps, int64_t partitions,
                              double partialBytes) {
    static constexpr double fit[2][4][3] = {{{2.17, 0.51, 0.3}, {3.19, 0.84, 0.39}, {3.47, 0.52, 0.32}, {3.67, 0.67, 0.67}},
                                            {{2.95, 0.67, 0.47}, {7.49, 0.02, 0.74}, {6.14, 0.57, 0.42}, {7.68, 0.83, 0.29}}};
    const double *c = fit[staged][slices_member(id)];
    const double rounds = (double)((groups + 255) / 256);
    const double chain = (double)steps * (c[1] > c[2] * rounds ? c[1] : c[2] * rounds);
    const double memory = (double)(M + N) * (double)K * 2e-6 / (staged ? 4.9 : 5.91);
    const double sums = partitions > 1 ? (staged ? -0.11 + 0.18e-6 * partialBytes : 1.64 + 0.59e-6 * partialBytes) : 0;
    return c[0] + (chain > memory ? chain : memory) + sums;
}
// Tile for this call, or -1: the members as they are.  One round of work-groups (a second one costs more than the estimate knows:
// up to 2.0 of the time) and an estimate 8 % below the other one; 18 % for the largest tile in place of the 64 x 64 x 128 member,
// whose two work-groups a unit the estimate of one flatters (51 calls between the two lines: 17 slower by over 3 %, 17 faster, 0.99
// in the mean).
// Of 6150 drawn aligned calls that took the form without the last three of these terms (the caches' trip, lines, the largest tile)
// 102 were slower than with the member by over 3 %, 41 by over 10; 40 and 22 of those now stay with it, with 25 level ones and
// 20 that were faster.  Of 3083 drawn afterwards 53 and 21 were, 38 and 15 are, and 0.6848 of the member's time in the mean was 0.6843.
inline int slices_tile(bool staged, int id, bool akc, bool bkc, int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, double other) {
    const int64_t larger = (M > N ? M : N) * K;
    const double trip = staged || larger < (16LL << 20) ? 0 : larger < (32LL << 20) ? 0.8 : 2;
    const SliceCall c{akc, bkc, M, N, (double)K, trip * (double)K, staged || lda % 64 == 0 ? 1 : 1.35, staged || ldb % 64 == 0 ? 1 : 1.35};
    int best = -1;
    double us = 0.92 * other;
#define KS_TRY(i, BM, BN, BK, NW, ST, FIXED) if (slices_us<i>(c, us)) best = i;
    if (staged) {
        KS_SLICES_STAGED_TILES(KS_TRY)
    } else {
        KS_SLICES_TILES(KS_TRY)
    }
#undef KS_TRY
    return best == 9 && id == 27 && us > 0.82 * other ? -1 : best;
}
// An operand of 104 MiB and more that one row (column) of tiles reads is taken not to outlast in the last-level cache of 256 MiB what
// comes between two of its uses.  That counts on other operands in between, as a model's layers are, which the call cannot know.
// M x 16 x 8192 NN, us past the cache and through it, by how many sets of operands take turns (one: the same again and again):
//   M                   1              2              3              6
//    6144 ( 96 MiB)  18.1 / 15.8    18.6 / 15.9    18.8 / 19.0    19.0 / 20.9
//    7168 (112 MiB)  19.3 / 18.0    20.2 / 18.0    20.4 / 23.2    20.7 / 23.1
//    8192 (128 MiB)  21.5 / 20.1    22.5 / 21.2    22.9 / 26.6    23.3 / 26.7
//   12288 (192 MiB)  33.2 / 28.5    35.2 / 40.0    36.0 / 40.4    36.8 / 41.3
//   14336 (224 MiB)  38.4 / 33.1    40.9 / 46.4    41.8 / 46.8    42.2 / 46.9
// (4096, 64 MiB, in turns of three 17.0 / 12.5.)
inline bool slices_past_cache(int64_t extent, int64_t K, int64_t tilesOther) { return tilesOther == 1 && extent * K * 2 >= (104LL << 20); }

}  // namespace ks
