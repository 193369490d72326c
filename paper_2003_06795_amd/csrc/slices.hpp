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
struct SliceTile {
    int bm, bn, bk, waves, stages;
    double fixed;
};
constexpr SliceTile kSliceTiles[] = {
#define KS_ROW(i, BM, BN, BK, NW, ST, FIXED) {BM, BN, BK, NW, ST, FIXED},
    KS_SLICES_TILES(KS_ROW)
#undef KS_ROW
};
constexpr int kSliceTileCount = sizeof(kSliceTiles) / sizeof(kSliceTiles[0]);

// variant: 1 bkc, 2 akc, 16 binary16; stream: which operands are loaded past the last-level cache
void launch_bf16_slices(int tile, const GemmParams &p, int grid, int variant, int stream, hipStream_t s);

// us per 1024 of K that a compute unit's memory pipe takes for one operand of a tile of `extent` rows (of columns): a K-contiguous
// one by its bytes, of a row-contiguous one with less than 64 every k takes as long as a whole line
inline double slice_operand_us(int extent, bool kc, int bk) {
    if (bk == 32) return kc ? 2.09 : 2.03;            // (K-contiguous pieces of 64 bytes)
    return extent == 16 ? (kc ? 0.34 : 1.12) : extent == 32 ? (kc ? 0.66 : 1.33) : (kc ? 1.23 : 1.61);
}
// Estimate for one round of work-groups of tile `t`, us: the longest of a unit's memory pipe, memory (a row-contiguous operand in
// pieces of less than a line is fetched as often as a line has pieces), what a work-group has in flight of an operand that comes
// from memory behind its 2 us (one of 64 MiB and more: 2944 x 2 x 14976 NT 18.4 us by the member, 22.7 in 184 tiles of 16 x 16), and the
// L2s.
inline double slices_us(const SliceTile &t, bool akc, bool bkc, int64_t M, int64_t N, int64_t K) {
    const double k = (double)K, tiles = (double)((M + t.bm - 1) / t.bm) * (double)((N + t.bn - 1) / t.bn);
    const double pipe = k / 1024 * (slice_operand_us(t.bm, akc, t.bk) + slice_operand_us(t.bn, bkc, t.bk));
    const double memory = k * 2e-6 * ((double)M * (akc ? 1 : 64 / t.bm) + (double)N * (bkc ? 1 : 64 / t.bn)) / 5.99;
    const double l2 = tiles * (t.bm + t.bn) * k * 2e-6 / 17.02;
    const double latency = M * K >= (32LL << 20) || N * K >= (32LL << 20) ? 2.0 * k / (t.waves * (t.stages - 1) * t.bk) : 0;
    double longest = pipe > memory ? pipe : memory;
    longest = longest > l2 ? longest : l2;
    return t.fixed + (longest > latency ? longest : latency);
}
// The same for the member (id) that the call would run otherwise, `steps` K-steps in each of `groups` work-groups, 0 where the
// form does not stand in for it; partitions > 1: their sums are `partialBytes` and a second launch adds them.
inline double slices_other_us(int id, int64_t M, int64_t N, int64_t K, int64_t groups, int64_t steps, int64_t partitions,
                              double partialBytes) {
    const double *c = nullptr;
    static constexpr double k13[] = {2.17, 0.51, 0.3}, k27[] = {3.19, 0.84, 0.39}, k38[] = {3.47, 0.52, 0.32}, k39[] = {3.67, 0.67, 0.67};
    if (id == 13) c = k13;
    else if (id == 27) c = k27;
    else if (id == 38) c = k38;
    else if (id == 39) c = k39;
    if (!c) return 0;
    const double rounds = (double)((groups + 255) / 256);
    const double chain = (double)steps * (c[1] > c[2] * rounds ? c[1] : c[2] * rounds);
    const double memory = (double)(M + N) * (double)K * 2e-6 / 5.91;
    return c[0] + (chain > memory ? chain : memory) + (partitions > 1 ? 1.64 + 0.59e-6 * partialBytes : 0);
}
// Tile for this call, or -1: the members as they are.  One round of work-groups (a second one costs more than the estimate knows:
// up to 2.0 of the time), K from 512 on (below, level) and an estimate 8 % below the other one.
inline int slices_tile(bool akc, bool bkc, int64_t M, int64_t N, int64_t K, double other) {
    if (K < 512 || K % 64 != 0 || M > (1 << 24) || N > (1 << 24)) return -1;
    int best = -1;
    double us = 0.92 * other;
    for (int i = 0; i < kSliceTileCount; ++i) {
        const SliceTile &t = kSliceTiles[i];
        if (((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn) > 256) continue;
        const double x = slices_us(t, akc, bkc, M, N, K);
        if (x < us) { us = x; best = i; }
    }
    return best;
}
// An operand of 96 MiB and more that one row (column) of tiles reads does not outlast in the last-level cache of 256 MiB what comes
// between two of its uses: 6000 x 16 x 8192 (94 MiB) is level, 8192 x 16 x 8192 0.87 of the time, 4096 x 16 x 8192 1.36.
inline bool slices_past_cache(int64_t extent, int64_t K, int64_t tilesOther) { return tilesOther == 1 && extent * K * 2 >= (96LL << 20); }

}  // namespace ks
