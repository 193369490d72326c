// Runtime kernel selection (paper Section IV): a decision tree deployed as integer comparisons, and beside
// the built-in trees the rules for what a count of tiles per compute unit, a few rows or columns or ragged sizes decide.
// Host only; no device access, no allocation.
#include "../../include/ks_gemm.h"

#include <limits.h>
#include <string.h>

#include "kept_set.inc"
#include "selector_table.inc"

namespace {

struct Deployed {
    ks_tree_node_t nodes[KS_MAX_TREE_NODES];
    int n;
    bool custom;
};
Deployed g_tree[2];

const ks_tree_node_t *builtin(int dtype, int *n) {
    if (dtype == KS_F32) {
        *n = (int)(sizeof(kTreeF32) / sizeof(kTreeF32[0]));
        return kTreeF32;
    }
    *n = (int)(sizeof(kTreeBf16) / sizeof(kTreeBf16[0]));
    return kTreeBf16;
}

const ks_tree_node_t *active(int dtype, int *n) {
    if (g_tree[dtype].custom) {
        *n = g_tree[dtype].n;
        return g_tree[dtype].nodes;
    }
    return builtin(dtype, n);
}

int64_t sat_mul(int64_t a, int64_t b) {
    if (a == 0 || b == 0) return 0;
    if (a > INT64_MAX / b) return INT64_MAX;
    return a * b;
}

// ---- the built-in trees and what they cannot follow --------------------------------------------
// The trees split on sizes; what a call costs steps with its tiles per compute unit, which no threshold of
// theirs can follow.  Where both sides were timed (operands rotated through three buffers) the choice is
// corrected, from the sizes alone: every caller of ks_select and every selecting entry point gets the same
// member, whatever the alignment of its operands, and whatever its scratch but for the rules that count on a K split
// (by_few_rows_or_columns): a call whose scratch does not hold the partitions gets what it would without them.  A caller's own
// tree is followed as it is.  (Whether the K-slices form then runs in place of a 16-bit member, slices.hpp, follows from alignment and
// scratch too.)
struct Tile {
    int id, bm, bn, bk;
};
constexpr Tile kTilesF32[] = {
#define KS_F32_INSTANCE(id, CORE, BM, BN, BK, P1, P2, SPLITK) {id, BM, BN, BK},
#include "instances.def"
#undef KS_F32_INSTANCE
};
constexpr Tile kTiles16[] = {
#define KS_BF16_INSTANCE(id, F, BM, BN, BK, WM, WN, STAGES, SPLITK) {id, BM, BN, BK},
#include "instances.def"
#undef KS_BF16_INSTANCE
};
template <int N>
constexpr bool tile_is(const Tile (&t)[N], int id, int bm, int bn, int bk) {
    return t[id].id == id && t[id].bm == bm && t[id].bn == bn && t[id].bk == bk;
}
// a member that a pruned library does not hold is not named by the full one either
constexpr int kKeptF32[] = KS_KEPT_F32;
constexpr int kKept16[] = KS_KEPT_BF16;
template <int N>
constexpr bool kept(const int (&list)[N], int id) {
    for (int i = 0; i < N; ++i)
        if (list[i] == id) return true;
    return false;
}
constexpr int kF32Large = 47, kF32Small = 28, k16Narrow = 23, k16TwoGroups = 47, k16OneGroup = 9;
constexpr int k16Columns = 13, k16ColumnsDeep = 38, k16Square = 27, k16SquareDeep = 39;
constexpr int k16Wide = 7, k16Large = 45;
constexpr int kF32ShortK = 23, kF32Halves = 41, kF32Tall = 15, kF32Sixteen = 38, kF32Half = 21, kF32GroupsLarge = 32, kF32Groups = 30;
static_assert(tile_is(kTilesF32, kF32Large, 128, 128, 32) && tile_is(kTilesF32, kF32Small, 64, 64, 16) &&
                  tile_is(kTiles16, k16Narrow, 128, 64, 64) && tile_is(kTiles16, k16TwoGroups, 128, 128, 128) &&
                  tile_is(kTiles16, k16OneGroup, 128, 128, 128) && tile_is(kTiles16, k16Columns, 64, 16, 128) &&
                  tile_is(kTiles16, k16ColumnsDeep, 64, 16, 128) && tile_is(kTiles16, k16Square, 64, 64, 128) &&
                  tile_is(kTiles16, k16SquareDeep, 64, 64, 128) && tile_is(kTiles16, k16Wide, 128, 128, 64) &&
                  tile_is(kTiles16, k16Large, 256, 256, 64) && tile_is(kTilesF32, kF32ShortK, 64, 64, 8) &&
                  tile_is(kTilesF32, kF32Halves, 32, 32, 32) && tile_is(kTilesF32, kF32Tall, 32, 64, 32) &&
                  tile_is(kTilesF32, kF32Sixteen, 16, 16, 32) && tile_is(kTilesF32, kF32Half, 32, 32, 16) &&
                  tile_is(kTilesF32, kF32GroupsLarge, 64, 64, 16) && tile_is(kTilesF32, kF32Groups, 32, 32, 32),
              "the rules below count the tiles of these members");

// fp32 128 x 128 -> 64 x 64.  A unit works through its tiles one after the other, so what counts is the fullest
//   unit: r128 quarters of large tiles against r64 small ones.
//   K < 1024, r64 <= 6/7 r128: 52 problems at 0.82 of the time (6272 x 704 x 576 79 -> 57 us, 3312 x 888 x 320 30 -> 24),
//     one of them slower (1.006); from 7/8 on also 1.10.
//   K <= 128 and a ragged last column of large tiles, which the pass over C decides: 60 more at 0.87 (17956 x 1067 x 15
//     29 -> 22 us, 14400 x 1147 x 45 38 -> 29), four of them slower by up to 1.056; with whole columns 1.10.
//   K >= 1024, where the large tiles may be shared out evenly among all units: only if padding to them costs a
//     fifth as well.  25 problems at 0.78, 0.73 without scratch (25088 x 288 x 1152 217 -> 180, 204800 x 33 x 1287 569 -> 358); at
//     less padding up to 1.34.
// 16-bit 128 x 64 -> 128 x 128 in two groups of waves: one round of large tiles that fills over half the device, whole
//   K-steps, K >= 2048.  2048^3 NT 27.8 -> 22.4 us, 1024 x 4096 x 4096 TN 46.4 -> 40.4; 22 problems at 0.86; rows of no
//   alignment 0.94 (2001 x 1999 x 3072 NT 35 -> 27, TT level); level at K = 1664, behind below 1024.
// 16-bit two groups of waves -> one, same tile: the last K-step half a one, which costs the two-group form branches
//   in every memory slot.  21 problems at 0.94 (2560 x 1280 x 1728 NT 20.5 -> 19.2 us), 0.97 where nothing is
//   aligned; not with both operands K-contiguous and a long K (1600 x 1216 x 5824 NT 45.7 -> 49.6).
int by_tiles_per_unit(int dtype, int id, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB) {
    if (batch != 1 || M <= 0 || N <= 0 || K <= 0 || M > (1 << 28) || N > (1 << 28)) return id;
    auto tiles = [&](int64_t e) { return ((M + e - 1) / e) * ((N + e - 1) / e); };
    const int64_t t128 = tiles(128);
    if (dtype == KS_F32) {
        if (id != kF32Large || !kept(kKeptF32, kF32Small)) return id;
        const int64_t t64 = tiles(64), r64 = (t64 + 255) / 256, r128 = 4 * ((t128 + 255) / 256);
        const bool small = K < 1024 ? 7 * r64 <= 6 * r128 || (K <= 128 && N % 128 != 0)
                                    : 4 * r64 <= 3 * r128 && 6 * t64 <= 20 * t128;
        return small ? kF32Small : id;
    }
    if (t128 <= 128 || t128 > 256) return id;
    if (id == k16Narrow && K % 128 == 0 && K >= 2048 && kept(kKept16, k16TwoGroups)) return k16TwoGroups;
    if (id == k16TwoGroups && K % 128 == 64 && (transA != 0 || transB == 0 || K <= 2048) && kept(kKept16, k16OneGroup))
        return k16OneGroup;
    return id;
}

// 16-bit products of a wide operand with a few columns or rows, one pass over the wide one.  The tables the tree was
//   trained on hold two such sizes, timed on operands that stay in the last-level cache.  With operands from memory
//   (three sets in turn; 7856 problems, the wide side and K in 1024 .. 16384, 1 to 128 on the other, whole and ragged sizes):
//   up to 16 columns: 64 x 16 tiles with three K-steps in flight for 64 x 64 ones, which load and multiply what does not
//     exist (1304 at 0.79: 8192 x 1 x 8192 NN 48 -> 35 us, 2048 x 4 x 16384 35 -> 19; behind by 3 - 9 % where both operands
//     are row-contiguous and whole, which keep the square tiles), and for the same tile with no K split from K = 1792 on
//     (322 at 0.65; below, 1.03 and more on every tenth).  The tree's other square member up to 32 columns (208 at 0.71).
//   up to 32 rows: 64 x 64 tiles for 64 x 16 ones, four times the work-groups over the same rows, and for three K-steps
//     in flight, which cost a resident work-group (1354 at 0.58: 6 x 6163 x 5041 NT 57 -> 28 us, 13 x 3909 x 12757 NN 39 ->
//     29; from 1536 columns on, below some at 1.15); for 64 x 16 without a split up to 16 rows and 8192 columns, K >= 2048 (160 at 0.59).
//   Those that gain by a K split stay with the tree's member in a call without scratch for it: unsplit, 27 is 1.07 - 1.32 times
//   as slow there as 38 and 13.
int by_few_rows_or_columns(int dtype, int id, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB,
                           bool scratch) {
    if (dtype == KS_F32 || batch != 1 || K < 1024) return id;
    if (M >= 1024 && N <= 32 && kept(kKept16, k16ColumnsDeep)) {
        const bool wholeTT = transA != 0 && transB != 0 && M % 8 == 0 && K % 8 == 0;
        if (N <= 16 && id == k16Square && !wholeTT) return k16ColumnsDeep;
        if (N <= 16 && id == k16Columns && K >= 1792 && scratch) return k16ColumnsDeep;
        if (id == k16SquareDeep && (N <= 16 || !wholeTT)) return k16ColumnsDeep;
        return id;
    }
    if (M <= 32 && N >= 1024 && K >= 2048 && kept(kKept16, k16Square)) {
        if (N >= 1536 && (id == k16SquareDeep || (id == k16ColumnsDeep && scratch))) return k16Square;
        if (id == k16Columns && M <= 16 && N < 8192 && scratch) return k16Square;
    }
    return id;
}

// Sizes that the tables hold few of or none (they are multiples of eight and were timed on cached operands): members
//   compared on 11491 drawn problems, whole and ragged, operands rotated through three sets.
// 16-bit, `ragged`: no leading dimension puts these sizes on the direct-to-LDS path as they are.  Where K alone is no whole
//   number of K-steps but a multiple of eight, NN, TN and TT run its whole steps there (dispatch.hip) and are not ragged: as
//   such they took 256 x 256 tiles for 128 x 128 at 1.03 of the time (16 drawn, worst 1.18: 5720 x 3176 x 1656 TN) and for
//   128 x 64 below 1.5e10 at 1.04 (8, worst 1.14).
//   128 x 64 -> 256 x 256 in two groups of waves, whose ragged operands are copied where there is scratch, once half the
//     device has such a tile: from 1.5e10 products on, ragged from 1.0e10: aligned 59 at 0.85 (worst 1.02), ragged 74 at 0.73,
//     0.94 without scratch (1.10).  With fewer tiles only a K split pays (0.84 with scratch, 1.16 without).  128 x 128 x 64 only
//     ragged, from 3e10 on and up to two rounds: 17 at 0.63, 0.89 without scratch (1.25); aligned 1.02.
//   64 x 64 -> 128 x 128 in two groups of waves, from 2.1e6 entries on, where half the device has a tile: 45 at 0.79 with
//     and without scratch (one at 1.3).
// fp32, `odd`: an operand whose rows are no multiple of four.
//   64 x 64 x 16 -> 64 x 64 x 8 up to K = 24, and 32 x 32 x 32 -> 64 x 64 x 8 up to K = 71, on large outputs: what a K-step holds
//     beyond K is loaded element by element and multiplied all the same (181 at 0.88, six over 1.03; 28 at 0.83).
//   members with two K groups -> 32 x 32 x 32: 41 at 0.88 where K is short, 40 at 0.89 where it is long.
//   batches: 32 columns or fewer on 32 x 64 tiles -> 32 x 32 (31 at 0.83, none slower); items that fill less than nine
//     tenths of their 16 x 16 tiles -> 32 x 32 (118 at 0.89, twelve over 1.03: 1.12); 32 x 32 x 16 -> 64 x 64 from 9036 of the
//     former on (24 at 0.88).
// A larger tile is taken where it fits: its padded output against that of the tile it replaces is limited.  Drawn again
//   (1017 problems of other seeds and wider ranges), time of the larger tile by that ratio, beyond the limit and up to it:
//   128 x 64 and 128 x 128 -> 256 x 256 1.25: 1.08 (74 problems, worst 2.08: 93709 x 62 x 2633), 0.82 (137, 1.18)
//   64 x 64 -> 128 x 128 1.15: 1.00 (90, worst 1.36: 152 x 18008 x 2640), 0.80 (48, 1.10)
//   32 x 32 x 32 -> 64 x 64 x 8 1.34: 1.03 (44, worst 1.49: 179963 x 20 x 59), 0.83 (96, 1.09)
//   batches 32 x 32 x 16 -> 64 x 64 1.25: 1.20 (72, worst 1.93: 82 x 21 x 65, 8910 of them), 0.84 (48, 1.09)
//   batches 16 x 16 -> 32 x 32 1.34: 1.03 (29, worst 1.25: 37 x 42 x 61), 0.84 (91, 1.10)
// Held out: 1860 problems of two later draws on which the rules act as they stand, time against the member replaced (count,
//   those over 1.03, worst): 256 x 256 for 128 x 64 ragged 0.75 (119, 4, 1.19), whole 0.84 (65, 2, 1.15); for 128 x 128 x 64 0.71 (114,
//   4, 1.06), level where nothing but K of NT is ragged (31, 8, 1.10); 128 x 128 for 64 x 64 0.79 (128, 3, 1.11); fp32 64 x 64 x 8 for
//   64 x 64 x 16 0.90 (64, 5, 1.12), for 32 x 32 x 32 0.83 (256, 15, 1.15); 32 x 32 x 32 for two K groups, short K 0.86 (64, 6, 1.13), long
//   0.92 (64, 7, 1.35: five rows, fewer than any problem the line was drawn from); batches in that order 0.87 (64, none), 0.84
//   (251, 16, 1.12), 0.83 (128, 1, 1.09).  Few rows or columns (by_few_rows_or_columns): 0.83, 0.71 and 0.72 for columns (64 each, 1.04), 0.61,
//   0.59 and 0.74 for rows (128, 128, 64; 1.14).
// leaf: what the tree says
int by_tile_fit(int dtype, int leaf, int id, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB) {
    if (M <= 0 || N <= 0 || K <= 0 || batch <= 0 || M > (1 << 28) || N > (1 << 28) || batch > (1 << 28)) return id;
    const double entries = (double)M * (double)N, products = entries * (double)K;
    auto padded = [&](int member) {
        const Tile &t = dtype == KS_F32 ? kTilesF32[member] : kTiles16[member];
        return (double)((M + t.bm - 1) / t.bm * t.bm) * (double)((N + t.bn - 1) / t.bn * t.bn);
    };
    auto fits = [&](int member, double limit) { return padded(member) <= limit * padded(id); };
    auto tiles = [&](int64_t e) { return (double)((M + e - 1) / e) * (double)((N + e - 1) / e); };
    if (dtype != KS_F32) {
        if (batch != 1) return id;
        const bool endOfK = K % 64 != 0 && (K % 8 != 0 || (transA == 0 && transB != 0));
        const bool ragged = endOfK || (transA != 0 && M % 8 != 0) || (transB == 0 && N % 8 != 0);
        const double large = tiles(256);
        if (kept(kKept16, k16Large) && large >= 128 && fits(k16Large, 1.25) &&
            ((id == k16Narrow && (products >= 1.5e10 || (ragged && products >= 1e10))) ||
             (id == k16Wide && ragged && products >= 3e10 && large < 512)))
            return k16Large;
        if (id == k16Square && kept(kKept16, k16TwoGroups) && tiles(128) >= 128 && entries >= 2.1e6 && fits(k16TwoGroups, 1.15))
            return k16TwoGroups;
        return id;
    }
    if (batch == 1) {
        const bool odd = (transA != 0 ? M : K) % 4 != 0 || (transB != 0 ? K : N) % 4 != 0;
        if (!odd) return id;
        if (kept(kKeptF32, kF32ShortK) && ((leaf == kF32Small && K <= 24 && entries >= 1 << 20) ||
                                           (id == kF32Halves && K <= 71 && entries >= 2.1e6 && fits(kF32ShortK, 1.34))))
            return kF32ShortK;
        if (kept(kKeptF32, kF32Halves) && ((id == kF32GroupsLarge && K < 576 && tiles(16) < 6038) ||
                                           (id == kF32Groups && K >= 1226 && (double)(M + N) * (double)K >= 1.65e6)))
            return kF32Halves;
        return id;
    }
    if (kept(kKeptF32, kF32Halves) &&
        ((id == kF32Tall && N <= 32) || (id == kF32Sixteen && M >= 17 && N >= 17 && entries < 0.9 * 256.0 * tiles(16) &&
                                         (M % 8 != 0 || N % 8 != 0 || K % 8 != 0) && fits(kF32Halves, 1.34))))
        return kF32Halves;
    if (id == kF32Half && tiles(32) * (double)batch >= 9036 && kept(kKeptF32, kF32Small) && fits(kF32Small, 1.25)) return kF32Small;
    return id;
}

}  // namespace

extern "C" int ks_features(int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB,
                           int64_t *out) {
    if (!out) return KS_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0 || batch < 0) return KS_ERR_INVALID_ARG;
    if ((transA != 0 && transA != 1) || (transB != 0 && transB != 1)) return KS_ERR_INVALID_ARG;
    out[0] = M;
    out[1] = N;
    out[2] = K;
    out[3] = batch;
    out[4] = transA;
    out[5] = transB;
    out[6] = sat_mul(M, N);
    out[7] = sat_mul(out[6], K);
    out[8] = M < N ? M : N;
    out[9] = M < N ? N : M;
    return KS_OK;
}

namespace ks {
// whether a rule that counts on a K split looks at these sizes (by_few_rows_or_columns): elsewhere scratch changes nothing below
bool split_decides(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch) {
    return dtype != KS_F32 && batch == 1 && K >= 1024 && ((M >= 1024 && N <= 32) || (M <= 32 && N >= 1024));
}
bool custom_tree(int dtype) { return g_tree[dtype == KS_F32 ? KS_F32 : KS_BF16].custom; }
// The member for these sizes; without scratch (for the partitions it takes) the rules that count on a K split are left out.
int select_member(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB, bool scratch) {
    if (dtype == KS_F16) dtype = KS_BF16;          // the fp16 form runs the 16-bit family with its tree
    if (dtype != KS_F32 && dtype != KS_BF16) return KS_ERR_INVALID_ARG;
    int64_t f[KS_NUM_FEATURES];
    const int rc = ks_features(M, N, K, batch, transA, transB, f);
    if (rc != KS_OK) return rc;
    int n = 0;
    const ks_tree_node_t *t = active(dtype, &n);
    int i = 0;
    // children always have larger indices than their parent, so the walk ends within n steps
    for (int step = 0; step < n && t[i].feature >= 0; ++step)
        i = f[t[i].feature] <= t[i].threshold ? t[i].left : t[i].right;
    if (t[i].feature >= 0) return KS_ERR_INVALID_ARG;
    if (g_tree[dtype].custom) return t[i].value;
    const int id = by_tiles_per_unit(dtype, t[i].value, M, N, K, batch, transA, transB);
    const int few = by_few_rows_or_columns(dtype, id, M, N, K, batch, transA, transB, scratch);
    return by_tile_fit(dtype, t[i].value, few, M, N, K, batch, transA, transB);
}
}  // namespace ks

extern "C" int ks_select(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB) {
    return ks::select_member(dtype, M, N, K, batch, transA, transB, true);
}

extern "C" int ks_set_selector(int dtype, const ks_tree_node_t *nodes, int n) {
    if (dtype != KS_F32 && dtype != KS_BF16) return KS_ERR_INVALID_ARG;
    if (n == 0) {
        g_tree[dtype].custom = false;
        return KS_OK;
    }
    if (!nodes || n < 0 || n > KS_MAX_TREE_NODES) return KS_ERR_INVALID_ARG;
    const int nk = ks_num_kernels(dtype);
    for (int i = 0; i < n; ++i) {
        if (nodes[i].feature < 0) {
            if (nodes[i].value < 0 || nodes[i].value >= nk) return KS_ERR_INVALID_ARG;
        } else {
            if (nodes[i].feature >= KS_NUM_FEATURES) return KS_ERR_INVALID_ARG;
            if (nodes[i].left <= i || nodes[i].left >= n) return KS_ERR_INVALID_ARG;
            if (nodes[i].right <= i || nodes[i].right >= n) return KS_ERR_INVALID_ARG;
        }
    }
    memcpy(g_tree[dtype].nodes, nodes, sizeof(ks_tree_node_t) * (size_t)n);
    g_tree[dtype].n = n;
    g_tree[dtype].custom = true;
    return KS_OK;
}

extern "C" int ks_get_selector(int dtype, ks_tree_node_t *nodes, int cap) {
    if (dtype != KS_F32 && dtype != KS_BF16) return KS_ERR_INVALID_ARG;
    int n = 0;
    const ks_tree_node_t *t = active(dtype, &n);
    if (!nodes || cap < n) return KS_ERR_INVALID_ARG;
    memcpy(nodes, t, sizeof(ks_tree_node_t) * (size_t)n);
    return n;
}

extern "C" const char *ks_status_string(int status) {
    switch (status) {
        case KS_OK: return "success";
        case KS_ERR_INVALID_ARG: return "invalid argument";
        case KS_ERR_UNSUPPORTED: return "unsupported size";
        case KS_ERR_LAUNCH: return "HIP launch failed or no device";
        case KS_ERR_WORKSPACE: return "split-K workspace missing or too small";
        default: return status > 0 ? "not a status (non-negative value)" : "unknown status";
    }
}
