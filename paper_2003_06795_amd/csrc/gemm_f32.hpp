// fp32 members of the tiled GEMM family (paper Section II).
//
// One kernel template; an instantiation fixes
//   BM x BN   work-group tile of C, staged operand tiles live in LDS (double buffered)
//   BK        K-step per stage (the paper's accumulator step, at work-group granularity)
//   CORE      inner-product engine:
//               FMA     each lane owns a TM x TN register tile and does outer-product FMAs;
//                       work-group = (BM/TM) x (BN/TN) lanes  (the paper's per-work-item tile)
//               MFMA16  each wave owns WM x WN built from 16x16x4 fp32 MFMA fragments
//               MFMA32  each wave owns WM x WN built from 32x32x2 fp32 MFMA fragments
//   P1 x P2   TM x TN for FMA, WM x WN for the MFMA cores
//   SPLIT     the instantiation is a split-K member: partial sums go to the workspace
//   AKC/BKC   whether op(A)/op(B) is K-contiguous in memory (A: transA == 0, B: transB == 1);
//             decides the coalescing direction of the global loads
//   LOADS     how a K-step is fetched (ks_common.hpp, TileLoader)
//
// LDS layout.  A row-contiguous operand: tile[k][m or n] with the row padded by 4 floats; all cores read "one k, many
// m/n", so rows of consecutive m/n are conflict-free for them.  A K-contiguous operand of the MFMA cores (K-steps of
// at least eight k with 32-wide and sixteen with 16-wide fragments): tile[m or n][k] as it comes from memory, in
// chunks of four k whose place in the row is XOR-swizzled by the row (F32Chunks).  A lane reads a chunk, four
// consecutive k of its row, and MFMA j of a group of four takes element j of both operands, so the sum over the
// group runs in another order than k's.  With [k][row] tiles for both, a K-contiguous operand took four times as many
// LDS instructions either way, which the matrix pipe's neighbours wait to issue: over the members in layouts NN / NT / TT
// and one to forty K-steps 0.97 of the time in the mean, 0.945 in NT (1024^3 NT 31.2 -> 28.8 us on 64 x 64 x 16, 4096^3 1051 -> 994
// on 128 x 128 x 32, 26.5 -> 23.4 on sixteen waves of 64 x 64 x 32; the balanced form of
// 64 x 64 x 32, 2000 x 2000 x 2048 162 -> 153, 640 x 640 x 4096 47.7 -> 46.0).
#pragma once
#include "ks_common.hpp"

namespace ks {

// Staging-register sets (K-steps in flight) as a function of the registers one set takes and the
// work-group size.  Measured on the small-problem workload: depth 4 gains 5 - 8 % for 8-register
// sets and 2 - 3 % for 16-register sets of four-wave work-groups, but costs 2 % for the eight-wave
// 128 x 128 x 32 tile, which already has two waves per SIMD to cover the latency; odd depths lose
// (the LDS buffer of a step is then no longer fixed inside the unrolled body).
#ifndef KS_F32_PREFETCH
#define KS_F32_PREFETCH(regs, threads) \
    ((regs) <= 8 || ((regs) <= 16 && (threads) <= 256) ? 4 : (regs) <= 32 ? 2 : 1)
#endif

// Waves per SIMD the register allocation must leave room for (0 = no demand).  The multi-tile
// forms keep the next tile's staging registers alive across the epilogue; the four-wave members
// with 64 x 32 wave tiles then drift a few registers past the budget of three waves per SIMD (168
// with the accumulators) that they met before, and lose a resident work-group; the eight-wave members
// need four.  The sixteen-wave 16x16 members without K groups hold two work-groups per compute unit with 64
// registers and would take 65 - 67 with both kinds of K-step in their loop.
#ifndef KS_F32_MIN_WAVES
#define KS_F32_MIN_WAVES(multi, core, bm, bn, bk, p1, p2, kw, loads)                                             \
    ((core) == CORE_MFMA16 && ((bm) / (p1)) * ((bn) / (p2)) == 16 && (kw) == 1 && (loads) == LOAD_STEPS ? 8 \
     : !(multi)                                                                                          ? 0 \
     : ((bm) / (p1)) * ((bn) / (p2)) <= 4                                                                ? 3 \
                                                                                                         : 4)
#endif
// The balanced persistent form counts on a fixed number of resident work-groups per compute unit:
// three of four waves (three per SIMD), which is what the plain form of that member reaches.
#ifndef KS_F32_SK_MIN_WAVES
#define KS_F32_SK_MIN_WAVES 3
#endif

enum { CORE_FMA = 0, CORE_MFMA16 = 1, CORE_MFMA32 = 2, CORE_DIRECT = 3, CORE_KSLICE = 4 };

// UNITS forms with fragments of four k that are told to leave room for eight waves per SIMD: by itself the sixteen-wave 64 x 64 x 32
// member takes 70 registers in NN and TT and loses its second work-group (2048 x 2048 x 96 NN 13.7 -> 16.6 us; with two
// staging sets instead of four, which spilled 16, 13.5), 32 x 32 x 16 66 in NT (2048 x 2048 x 1024 101 -> 110; 102 with 62).  Where they fit
// unasked the demand costs up to 6 % (32 x 32 x 16 in the other layouts) and 3 % (64 x 64 x 32 in NT).
constexpr bool f32_units_eight_waves(int core, int bm, int bn, int bk, int p1, int p2, int kw, bool akc, bool bkc, int loads) {
    return loads == LOAD_UNITS && core == CORE_MFMA16 && kw == 1 &&
           ((bm / p1) * (bn / p2) == 16 ? bk >= 32 && akc != bkc : bm == 32 && bn == 32 && bk == 16 && akc && bkc);
}

template <int CORE, int BM, int BN, int P1, int P2>
struct F32Shape {
    static constexpr int threads =
        CORE == CORE_FMA ? (BM / P1) * (BN / P2) : CORE == CORE_KSLICE ? 64 * P1 * (BM / P2) * (BN / P2) : 64 * (BM / P1) * (BN / P2);
    static constexpr int frag = CORE == CORE_MFMA16 ? 16 : 32;
};

// LDS place (in floats) of the four k of chunk c of tile row r: rows of BK floats, chunks XOR-swizzled by the row
template <int BK>
struct F32Chunks {
    static constexpr int CPR = BK / 4, RP = CPR >= 16 ? 1 : 16 / CPR;      // chunks per row; rows per 256 bytes
    __device__ __forceinline__ static int at(int r, int c) { return r * BK + 4 * (c ^ ((r / RP) & (CPR - 1))); }
};

// ---- global -> registers -> LDS staging of one ROWS x BK operand tile ------------------------
// KC:  memory is [row][k] (k contiguous);  !KC: memory is [k][row] (row contiguous).
// Units are W floats (four, or one in the ELEMENTS form) walked so that consecutive lanes touch consecutive
// addresses.  INNER = units along the contiguous direction, OUTER = the other direction.
// CHUNKS: the tile is [row][k] in swizzled chunks of four k.
//
// load() is for K-steps in which every unit may be read whole (whole_steps() of them): the rows of a
// K-contiguous operand end at or behind the step, or the step of a row-contiguous one ends before the
// last k (a unit that hangs over the right edge of row k then reads the beginning of row k + 1, and
// what it gets belongs to rows of C that do not exist).  Rows beyond `limit` are clamped to valid ones
// for the same reason.  There is no predicate and no per-lane address arithmetic: a 32-bit lane
// offset that stays the same for the whole tile on a scalar address that advances with K.
// load_edge() is for the steps that are left, as a rule the one that holds the end of K: it reads
// inside the matrix only, and k beyond the end read as zero.
// load_units() serves any step of the UNITS and ELEMENTS forms with one predicate per unit, none of which
// straddles an edge there.  A short K runs these: the code of both other kinds, up to four K-steps deep, costs
// it more than the predicates (944 x 40x52x52 17.2 against 14.5 us, 4096 x 64x64x64 62.5 against 53.8, 3056 x 704 x 16
// NT 8.4 against 7.4), while from about ten K-steps on the predicates are the slower ones (1024^3 NN 26.1 against
// 24.6 us, 25088 x 256 x 1152 151 against 146), but for the members named in ks_common.hpp.
//
// What load() is there for: the large members wait for the issue of their loads, not for memory (a matrix
// pipe kept busy by other waves holds up vector-memory issue), and four-byte loads took four times as
// many of them.  Against scalar loads of unaligned operands and predicated ones of aligned operands:
// 4095 x 3000 x 4089 NT 950 -> 805 us (TN 1020 -> 797), 1000^3 with padded rows NN 33.3 -> 26.2 us;
// aligned 4096^3 TN 1058 -> 1006 us, 1024^3 NN 26.0 -> 24.5 us, im2col 25088 x 256 x 1152 149 -> 144 us.
template <int ROWS, int BK, int NT, bool KC, int W, bool CHUNKS = false>
struct TileLoader {
    typedef float Unit __attribute__((ext_vector_type(W)));
    static constexpr int INNER = (KC ? BK : ROWS) / W;
    static constexpr int OUTER = KC ? ROWS : BK;
    static constexpr int UNITS = INNER * OUTER;
    static constexpr int ITERS = (UNITS + NT - 1) / NT;
    static constexpr int STRIDE = NT / INNER;                // outer distance of a thread's units
    // Row padding of the LDS tile.  A K-contiguous operand is written as four scalars to rows
    // k .. k+3; a wave's lanes then differ in k by multiples of 4 (BK/4 lanes) and in the row, and
    // land in 64 different banks when 4 * LDS_LD = 256/BK (mod 64), i.e. a padding of 64/BK floats.
    // One written along a row takes the padding of 4 that keeps its 16-byte writes aligned.  (Measured:
    // bank-conflict cycles of the 128 x 128 x 32 member fell to a third and the BK = 32 / 64 members gained
    // 2 - 20 % on long K; giving the lane groups of an MFMA read rows 4 or 8 apart instead of adjacent ones
    // changed nothing.)
    static constexpr int LDS_LD = ROWS + (KC && W == 4 ? (BK >= 64 ? 1 : 64 / BK) : 4);
    static constexpr int LDS_SIZE = CHUNKS ? ROWS * BK : BK * LDS_LD;
    static_assert(KC || W == 1 || LDS_LD % 4 == 0, "row-contiguous vector writes need 16-byte alignment");
    static_assert(INNER <= NT && NT % INNER == 0, "walk");

    // byte offsets of a thread's units from the tile origin (row0, first k of the step); the units of a
    // row-contiguous operand differ by whole k rows, which the scalar address takes
    struct Plan {
        unsigned off[KC ? ITERS : 1];
        __device__ __forceinline__ void init(long long ld, int row0, int limit, int tid) {
#pragma unroll
            for (int it = 0; it < (KC ? ITERS : 1); ++it) {
                const int inner = tid % INNER, outer = tid / INNER + it * STRIDE;
                if constexpr (KC)
                    off[it] = ((unsigned)(min(row0 + outer, limit - 1) - row0) * (unsigned)ld + inner * W) * 4u;
                else
                    off[it] = (outer * (unsigned)ld + (row0 + inner * W < limit ? inner * W : 0)) * 4u;
            }
        }
    };

    Unit reg[ITERS];

    __device__ __forceinline__ static bool has(int tid, int it) {
        return UNITS % NT == 0 || tid / INNER + it * STRIDE < OUTER;
    }

    // leading K-steps of [kBegin, kEnd) that load() may take (lane offsets fit 32 bits below 2^22).  A unit that
    // hangs over the edge of row k reaches three elements beyond it, which lie inside the matrix while
    // (K - 1 - k) ld >= 3: all but the last row, or the last two or three where rows are that short.
    __device__ __forceinline__ static int whole_steps(long long ld, int limit, int K, int kBegin, int kEnd) {
        if (ld > (1LL << 22)) return 0;
        if (KC || (limit & 3) == 0) return max((kEnd - kBegin) / BK, 0);
        return max((min(kEnd, K - (ld >= 3 ? 1 : ld == 2 ? 2 : 3)) - kBegin) / BK, 0);
    }

    // tile: address of the tile origin at this K-step (the same for all lanes)
    __device__ __forceinline__ void load(const Plan &plan, const float *tile, long long ld, int tid) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const char *t = reinterpret_cast<const char *>(tile + (KC ? 0 : it * STRIDE * ld));
            if (has(tid, it)) reg[it] = load_float4_any(t + plan.off[KC ? it : 0]);
        }
    }

    // any step where no unit straddles an edge of the matrix: rows and k beyond it read as zero
    __device__ __forceinline__ void load_units(const float *base, long long ld, int row0, int limit, int k0, int kEnd,
                                               int tid) {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int inner = tid % INNER, outer = tid / INNER + it * STRIDE;
            const int row = row0 + (KC ? outer : inner * W), k = k0 + (KC ? inner * W : outer);
            const float *src = KC ? base + (long long)row * ld + k : base + (long long)k * ld + row;
            Unit v = 0.f;
            if (has(tid, it) && row < limit && k < kEnd) {
                if constexpr (W == 4) v = load_float4_any(src);
                else v[0] = *src;
            }
            reg[it] = v;
        }
    }

    // clear() goes before the load_edge() of both operands: zeros that the compiler writes between the
    // loads make it wait for those in flight.
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            reg[it] = floatx4{0.f, 0.f, 0.f, 0.f};
            asm volatile("" : "+v"(reg[it]));
        }
    }
    __device__ __forceinline__ void load_edge(const float *base, long long ld, int row0, int limit, int k0, int kEnd,
                                              int tid) {
        // (the addresses are recomputed here: the compiler would otherwise keep them in registers
        // across the K loop)
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            const int inner = tid % INNER, outer = tid / INNER + it * STRIDE;
            const int row = KC ? min(row0 + outer, limit - 1) : row0 + inner * W;
            const int k = KC ? k0 + inner * W : k0 + outer;
            const int n = !has(tid, it) ? 0 : KC ? kEnd - k : k < kEnd ? limit - row : 0;   // elements that exist
            const float *src = KC ? base + (long long)row * ld + k : base + (long long)k * ld + row;
            if (n >= W) {
                reg[it] = load_float4_any(src);
            } else {
#pragma unroll
                for (int e = 0; e < W - 1; ++e)
                    if (e < n) reg[it][e] = src[e];
            }
        }
    }

    // four consecutive k, from k on, of tile row `row`
    __device__ __forceinline__ static floatx4 read(const float *lds, int row, int k) {
        if constexpr (CHUNKS) return *reinterpret_cast<const floatx4 *>(lds + F32Chunks<BK>::at(row, k / 4));
        floatx4 v;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = lds[(k + j) * LDS_LD + row];
        return v;
    }

    __device__ __forceinline__ void store(float *lds, int tid) const {
#pragma unroll
        for (int it = 0; it < ITERS; ++it) {
            if (!has(tid, it)) continue;
            const int inner = tid % INNER, outer = tid / INNER + it * STRIDE;
            const int r = KC ? outer : inner * W;
            const int k = KC ? inner * W : outer;
            if constexpr (CHUNKS) {
                *reinterpret_cast<floatx4 *>(lds + F32Chunks<BK>::at(r, inner)) = reg[it];
            } else if constexpr (KC || W == 1) {
#pragma unroll
                for (int j = 0; j < W; ++j) lds[(k + j) * LDS_LD + r] = reg[it][j];
            } else {
                *reinterpret_cast<floatx4 *>(lds + k * LDS_LD + r) = reg[it];
            }
        }
    }
};

// The tiles and K-steps of one work-group of the balanced persistent form (SK below): body(tile, first K-step, last K-step + 1,
// K-steps of a tile, work-group, whether it is the head of the share of left-over tiles) for each.  Everything that describes
// the share is the same for all lanes; the integer divisions run on the vector unit, so their results are moved
// to scalar registers explicitly.
template <int BK, class Body>
__device__ __forceinline__ void sk_for_each_tile(const GemmParams &p, Body body) {
    auto uni = [](long long v) -> long long {
        const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(unsigned long long)v);
        const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)v >> 32));
        return (long long)(((unsigned long long)hi << 32) | lo);
    };
    const unsigned lw = (unsigned)__builtin_amdgcn_readfirstlane((int)logical_of_block());
    const long long groups = (long long)gridDim.x;
    const int nkT = (p.K + BK - 1) / BK;
    const long long units = (long long)p.skTailTiles * nkT;
    const long long ub = uni(sk_share_begin(lw, units, groups)), ue = uni(sk_share_begin(lw + 1, units, groups));
    const long long t0 = uni(ub / nkT);                      // first left-over tile of the share
    const int r0 = (int)(ub - t0 * nkT);                      // and the K-step it starts at
    const int tailSegs = ue > ub ? (int)(uni((ue - 1) / nkT) - t0) + 1 : 0;
    const int nSeg = p.skRounds + tailSegs;
    for (int sg = 0; sg < nSeg; ++sg) {
        unsigned logical;
        int ks0 = 0, ks1 = nkT;
        if (sg < p.skRounds) {
            logical = (unsigned)sg * (unsigned)groups + lw;
        } else {
            const long long t = t0 + (sg - p.skRounds);
            logical = (unsigned)p.skRounds * (unsigned)groups + (unsigned)t;
            ks0 = sg == p.skRounds ? r0 : 0;
            ks1 = (int)min((long long)nkT, ue - t * nkT);
        }
        TileCoord tc = tile_of_logical(p, logical);
        tc.batch = __builtin_amdgcn_readfirstlane(tc.batch);
        tc.tm = __builtin_amdgcn_readfirstlane(tc.tm);
        tc.tn = __builtin_amdgcn_readfirstlane(tc.tn);
        tc.split = 0;
        body(tc, ks0, ks1, nkT, lw, sg == p.skRounds);
    }
}

// raw accumulators of 32x32 fragments, in register order: float4 unit (wave, i, j, chunk) of lane l
template <int FM, int FN, class Acc>
__device__ __forceinline__ void store_units32(floatx4 *units, int wave, int lane, const Acc &acc) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                units[(((wave * FM + i) * FN + j) * 4 + c) * 64 + lane] =
                    floatx4{acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
}
// ... of a part of a tile in the balanced form: at most two per work-group, the head and the tail of its share
template <int BM, int BN, int FM, int FN, class Acc>
__device__ __forceinline__ void sk_store_part(const GemmParams &p, unsigned group, bool head, int wave, int lane, const Acc &acc) {
    store_units32<FM, FN>(reinterpret_cast<floatx4 *>(p.ws) + ((long long)group * 2 + (head ? 0 : 1)) * (BM * BN / 4), wave, lane, acc);
}

// Sums the accumulators of the K groups in group order, from float4 units [group][wave][i][j][chunk][lane] in LDS that are
// dealt out over all threads, and stores the tile at (row, col).  FRG: fragment edge, CH: chunks of a fragment and lane.
template <bool SPLIT, int FRG, int CH, int FM, int FN, int P1, int P2, int BN, int NT, int KW>
__device__ __forceinline__ void store_sum_of_groups(const floatx4 *part, const GemmParams &p, const TileCoord &tc, float *Cb, int row, int col) {
    constexpr int UNITS = (NT / 64) * FM * FN * CH * 64;
    const OutTarget o = out_target<SPLIT>(p, tc, Cb);
    for (int u = (int)threadIdx.x; u < UNITS; u += NT * KW) {
        floatx4 sum = part[u];
#pragma unroll
        for (int g = 1; g < KW; ++g) sum += part[g * UNITS + u];
        const int ul = u & 63;
        int q = __builtin_amdgcn_readfirstlane(u >> 6);
        const int c = q % CH; q /= CH;
        const int j = q % FN; q /= FN;
        const int i = q % FM;
        const int w = q / FM;
        const int fr0 = row + (w / (BN / P2)) * P1 + i * FRG, fc0 = col + (w % (BN / P2)) * P2 + j * FRG;
        const bool full = fr0 + FRG <= o.M && fc0 + FRG <= o.N;
        const float v[4] = {sum[0], sum[1], sum[2], sum[3]};
        if constexpr (FRG == 16)
            store_lane_column<SPLIT, 4>(o, fr0 + 4 * (ul >> 4), fc0 + (ul & 15), full, v, [](int e) { return e; });
        else
            store_lane_column<SPLIT, 4>(o, fr0 + 8 * c + 4 * (ul >> 5), fc0 + (ul & 31), full, v, [](int e) { return e; });
    }
}

// KW > 1 (MFMA cores): the work-group holds KW groups of waves, each a complete copy of the
// BM x BN wave arrangement with its own LDS stages, and each takes one slice of the work-group's
// K range (rounded to whole K-steps).  The groups run the same number of K-steps in lock-step (a
// short slice pads with zero tiles), then add their accumulators through LDS in group order.
// More waves per compute unit for the same number of tiles, without a workspace.
//
// MULTI (members for which f32_multi_tile holds, never split-K): the work-group walks
// GemmParams::tilesPerWG consecutive logical tiles.  The single-tile form of the same member is a
// separate instantiation: the flattened loop costs it about 6 % on ordinary shapes.
//
// SK (32x32 MFMA members, single K group, never split-K): the balanced persistent form.  The launch
// holds a fixed number of work-groups (a few per compute unit, all resident at once).  Each first
// computes GemmParams::skRounds whole tiles, then an equal share of the K-steps of the tiles that
// are left over when the tile count is not a multiple of the work-group count: those tiles are
// flattened into one sequence of (tile, K-step) units and cut into contiguous shares, so every
// compute unit gets the same number of K-steps however unevenly the tiles divide.  A share that
// covers a whole tile is written to C as usual; a share that covers part of a tile goes to the
// workspace as a raw accumulator tile (at most two per work-group: the head and the tail of its
// share), and gemm_f32_sk_fixup_kernel adds the parts of every divided tile in K order and applies
// the epilogue.  No work-group waits for another, so there is nothing to deadlock on.
template <int CORE, int BM, int BN, int BK, int P1, int P2, bool SPLIT, bool AKC, bool BKC,
          int LOADS, int KW = 1, bool MULTI = false, bool SK = false>
__global__ __launch_bounds__((F32Shape<CORE, BM, BN, P1, P2>::threads * KW), (SK ? KS_F32_SK_MIN_WAVES : f32_units_eight_waves(CORE, BM, BN, BK, P1, P2, KW, AKC, BKC, LOADS) ? 8 : KS_F32_MIN_WAVES(MULTI, CORE, BM, BN, BK, P1, P2, KW, LOADS))) void gemm_f32_kernel(
    const GemmParams p) {
    static_assert(LOADS == LOAD_STEPS || !(MULTI || SK), "persistent forms");
    static_assert(!MULTI || (f32_multi_tile(CORE, BM, BN, P1, P2, KW) && !SPLIT), "multi-tile form");
    static_assert(!SK || (CORE == CORE_MFMA32 && KW == 1 && !SPLIT && !MULTI), "balanced persistent form");
    using Shape = F32Shape<CORE, BM, BN, P1, P2>;
    constexpr int NT = Shape::threads;                        // threads of one group
    static_assert(KW == 1 || CORE != CORE_FMA, "K groups need an MFMA core");
    constexpr int W = LOADS == LOAD_ELEMENTS ? 1 : 4;
    constexpr int FR = Shape::frag, KV = 4 * (64 / FR);       // KV: k of a substep of whole chunks
    // groups of four k to a lane: the order of the sums, the same in every load form
    constexpr bool BY_FOUR = CORE != CORE_FMA && BK % KV == 0 && (AKC || BKC);
    constexpr bool CHA = BY_FOUR && W == 4 && AKC, CHB = BY_FOUR && W == 4 && BKC;
    using LoaderA = TileLoader<BM, BK, NT, AKC, W, CHA>;
    using LoaderB = TileLoader<BN, BK, NT, BKC, W, CHB>;
    constexpr int LDA = LoaderA::LDS_LD, LDB = LoaderB::LDS_LD;
    __shared__ __attribute__((aligned(1024))) float AsAll[KW][2][LoaderA::LDS_SIZE];
    __shared__ __attribute__((aligned(1024))) float BsAll[KW][2][LoaderB::LDS_SIZE];

    const int grp = KW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int tid = KW == 1 ? (int)threadIdx.x : (int)threadIdx.x % NT;
    float (*As)[LoaderA::LDS_SIZE] = AsAll[grp];
    float (*Bs)[LoaderB::LDS_SIZE] = BsAll[grp];
    // the (first) tile of this work-group
    const TileCoord tc = MULTI && !p.grid3d ? tile_of_logical(p, logical_of_block() * (unsigned)p.tilesPerWG)
                                            : tile_of_block(p);
    const int row0 = __builtin_amdgcn_readfirstlane(tc.tm) * BM, col0 = __builtin_amdgcn_readfirstlane(tc.tn) * BN;
    const float *Ab = static_cast<const float *>(p.A) + (long long)tc.batch * p.strideA;
    const float *Bb = static_cast<const float *>(p.B) + (long long)tc.batch * p.strideB;
    float *Cb = p.C + (long long)tc.batch * p.strideC;
    const int kLo = tc.split * p.kChunk, kHi = min(p.K, kLo + p.kChunk);
    const int slice = KW == 1 ? p.kChunk : ((((kHi - kLo) + KW - 1) / KW + BK - 1) / BK) * BK;
    const int kBegin = kLo + grp * slice;
    const int kEnd = min(kHi, kBegin + slice);               // may lie below kBegin: an empty slice
    const int nk = (min(slice, kHi - kLo) + BK - 1) / BK;     // steps of the longest slice, for all groups

    // K-steps in flight between global memory and LDS (each in its own set of staging registers):
    // small tiles are latency-bound - few waves per compute unit, short MFMA runs per K-step - and
    // afford several; large tiles hide the latency behind their MFMAs and keep the registers.
    constexpr int STAGE_REGS = (LoaderA::ITERS + LoaderB::ITERS) * W;
    // (sixteen waves that must fit 64 registers: four sets beside fragments of four k spilled 4 - 16)
    constexpr bool TIGHT = (KS_F32_MIN_WAVES(MULTI, CORE, BM, BN, BK, P1, P2, KW, LOADS) == 8 ||
                            f32_units_eight_waves(CORE, BM, BN, BK, P1, P2, KW, AKC, BKC, LOADS)) && (CHA || CHB) && BK >= 32;
    constexpr int PF = TIGHT ? 2 : KS_F32_PREFETCH(STAGE_REGS, NT);
    LoaderA la[PF];
    LoaderB lb[PF];
    typename LoaderA::Plan pa;
    typename LoaderB::Plan pb;
    // one K-step, from k0 on, of the tile at (r, c) that pa and pb describe
    auto load_step = [&](LoaderA &a, LoaderB &b, const float *A, const float *B, int r, int c, int k0, int kE, bool whole) {
        const float *at = AKC ? A + (long long)r * p.lda + k0 : A + (long long)k0 * p.lda + r;
        const float *bt = BKC ? B + (long long)c * p.ldb + k0 : B + (long long)k0 * p.ldb + c;
        if constexpr (LOADS != LOAD_STEPS) {
            a.load_units(A, p.lda, r, p.M, k0, kE, tid);
            b.load_units(B, p.ldb, c, p.N, k0, kE, tid);
        } else if (whole) {
            a.load(pa, at, p.lda, tid);
            b.load(pb, bt, p.ldb, tid);
        } else {
            a.clear();
            b.clear();
            a.load_edge(A, p.lda, r, p.M, k0, kE, tid);
            b.load_edge(B, p.ldb, c, p.N, k0, kE, tid);
        }
    };
    auto whole_steps = [&](int kB, int kE) {
        return min(LoaderA::whole_steps(p.lda, p.M, p.K, kB, kE), LoaderB::whole_steps(p.ldb, p.N, p.K, kB, kE));
    };

    // accumulators
    constexpr int FM = CORE == CORE_FMA ? 1 : P1 / FR, FN = CORE == CORE_FMA ? 1 : P2 / FR;
    float accF[CORE == CORE_FMA ? P1 : 1][CORE == CORE_FMA ? P2 : 1];
    floatx4 acc16[CORE == CORE_MFMA16 ? FM : 1][CORE == CORE_MFMA16 ? FN : 1];
    floatx16 acc32[CORE == CORE_MFMA32 ? FM : 1][CORE == CORE_MFMA32 ? FN : 1];
    if constexpr (CORE == CORE_FMA) {
#pragma unroll
        for (int i = 0; i < P1; ++i)
#pragma unroll
            for (int j = 0; j < P2; ++j) accF[i][j] = 0.f;
    } else if constexpr (CORE == CORE_MFMA16) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) acc16[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc32[i][j][e] = 0.f;
    }

    // lane -> sub-tile origin inside the work-group tile
    const int lane = tid & 63, wave = tid >> 6;
    int subM, subN;
    if constexpr (CORE == CORE_FMA) {
        subM = (tid / (BN / P2)) * P1;
        subN = (tid % (BN / P2)) * P2;
    } else {
        subM = (wave / (BN / P2)) * P1;
        subN = (wave % (BN / P2)) * P2;
    }

    // one K-step of MFMAs / FMAs on a landed LDS stage
    auto compute_step = [&](const float *as, const float *bs) {
        if constexpr (CORE == CORE_FMA) {
#pragma unroll
            for (int kk = 0; kk < BK; ++kk) {
                float a[P1], b[P2];
#pragma unroll
                for (int i = 0; i < P1; ++i) a[i] = as[kk * LDA + subM + i];
#pragma unroll
                for (int j = 0; j < P2; ++j) b[j] = bs[kk * LDB + subN + j];
#pragma unroll
                for (int i = 0; i < P1; ++i)
#pragma unroll
                    for (int j = 0; j < P2; ++j) accF[i][j] = fmaf(a[i], b[j], accF[i][j]);
            }
        } else if constexpr (BY_FOUR) {
            // a lane holds four consecutive k of its row, MFMA j of a group of four consumes element j
#pragma unroll
            for (int kk = 0; kk < BK; kk += KV) {
                const int g = lane / FR, r = lane % FR;
                floatx4 a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = LoaderA::read(as, subM + i * FR + r, kk + 4 * g);
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = LoaderB::read(bs, subN + j * FR + r, kk + 4 * g);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j) {
                            if constexpr (CORE == CORE_MFMA16)
                                acc16[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc16[i][j], 0, 0, 0);
                            else
                                acc32[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc32[i][j], 0, 0, 0);
                        }
            }
        } else if constexpr (CORE == CORE_MFMA16) {
            // 16x16x4: lane l feeds A[l%16][l/16] and B[l/16][l%16]
#pragma unroll
            for (int kk = 0; kk < BK; kk += 4) {
                const int kr = kk + (lane >> 4);
                float a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = as[kr * LDA + subM + i * 16 + (lane & 15)];
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = bs[kr * LDB + subN + j * 16 + (lane & 15)];
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc16[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc16[i][j], 0, 0, 0);
            }
        } else {
            // 32x32x2: lane l feeds A[l%32][l/32] and B[l/32][l%32]
#pragma unroll
            for (int kk = 0; kk < BK; kk += 2) {
                const int kr = kk + (lane >> 5);
                float a[FM], b[FN];
#pragma unroll
                for (int i = 0; i < FM; ++i) a[i] = as[kr * LDA + subM + i * 32 + (lane & 31)];
#pragma unroll
                for (int j = 0; j < FN; ++j) b[j] = bs[kr * LDB + subN + j * 32 + (lane & 31)];
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc32[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc32[i][j], 0, 0, 0);
            }
        }
    };

    if constexpr (MULTI) {
        // The work-group walks nTiles consecutive logical tiles as ONE sequence of K-steps: the
        // loads run PF steps ahead of the MFMAs across tile boundaries, so the first steps of the
        // next tile are requested before the finished tile's C is stored (the vector memory path
        // of a compute unit is in order: loads issued behind 64 KB of stores to a busy HBM wait
        // for them), and tiles after the first pay no work-group launch and no pipeline fill.
        // All tiles of a launch with tilesPerWG > 1 share one K range (the host grants it only
        // without split-K); a range without steps still runs one step of zero tiles.
        unsigned firstTile = 0;
        int nTiles = 1;
        if (!p.grid3d) {
            const unsigned total = (unsigned)p.tilesM * (unsigned)p.tilesN * (unsigned)(p.batch * p.splitK);
            firstTile = logical_of_block() * (unsigned)p.tilesPerWG;
            nTiles = (int)min((unsigned)p.tilesPerWG, total - firstTile);
        }
        const int nkT = max(nk, 1);
        const int G = nTiles * nkT;
        // load stream
        TileCoord tcL = tc;
        int iL = 0, kL = 0, rowL = row0, colL = col0;
        const float *AbL = Ab, *BbL = Bb;
        pa.init(p.lda, rowL, p.M, tid);
        pb.init(p.ldb, colL, p.N, tid);
        const int full = whole_steps(kBegin, kEnd);
        auto issue_load = [&](LoaderA &a, LoaderB &b) {
            load_step(a, b, AbL, BbL, rowL, colL, kBegin + kL * BK, kEnd, kL < full);
            if (++kL == nkT) {
                kL = 0;
                if (++iL < nTiles) {
                    tcL = tile_of_logical(p, firstTile + (unsigned)iL);
                    rowL = __builtin_amdgcn_readfirstlane(tcL.tm) * BM; colL = __builtin_amdgcn_readfirstlane(tcL.tn) * BN;
                    AbL = static_cast<const float *>(p.A) + (long long)tcL.batch * p.strideA;
                    BbL = static_cast<const float *>(p.B) + (long long)tcL.batch * p.strideB;
                    pa.init(p.lda, rowL, p.M, tid);
                    pb.init(p.ldb, colL, p.N, tid);
                }
            }
        };
        // compute stream
        TileCoord tcC = tc;
        int iC = 0, kC = 0;
#pragma unroll
        for (int d = 0; d < PF; ++d)
            if (d < G) issue_load(la[d], lb[d]);
        la[0].store(As[0], tid);
        lb[0].store(Bs[0], tid);
        __syncthreads();
        for (int g0 = 0; g0 < G; g0 += PF) {
#pragma unroll
            for (int u = 0; u < PF; ++u) {
                const int g = g0 + u;
                if (g >= G) break;
                const int cur = g & 1;
                if (g + PF < G) issue_load(la[u], lb[u]);
                compute_step(As[cur], Bs[cur]);
                if (g + 1 < G) {
                    la[(u + 1) % PF].store(As[cur ^ 1], tid);
                    lb[(u + 1) % PF].store(Bs[cur ^ 1], tid);
                }
                if (++kC == nkT) {
                    kC = 0;
                    float *Cc = p.C + (long long)tcC.batch * p.strideC;
                    write_tile_mfma32_lean<SPLIT, FM, FN>(p, tcC, Cc, tcC.tm * BM + subM, tcC.tn * BN + subN, lane, acc32);
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j)
#pragma unroll
                            for (int e = 0; e < 16; ++e) acc32[i][j][e] = 0.f;
                    if (++iC < nTiles) tcC = tile_of_logical(p, firstTile + (unsigned)iC);
                }
                __syncthreads();
            }
        }
        return;
    }

    if constexpr (SK) {
        sk_for_each_tile<BK>(p, [&](const TileCoord &tcS, int ks0, int ks1, int nkT, unsigned group, bool head) {
            const int rowS = tcS.tm * BM, colS = tcS.tn * BN;
            const float *AbS = static_cast<const float *>(p.A) + (long long)tcS.batch * p.strideA;
            const float *BbS = static_cast<const float *>(p.B) + (long long)tcS.batch * p.strideB;
            const int kB = ks0 * BK, kE = min(p.K, ks1 * BK), nkS = ks1 - ks0;
            pa.init(p.lda, rowS, p.M, tid);
            pb.init(p.ldb, colS, p.N, tid);
            const int full = whole_steps(kB, kE);
            // every staging set is (re)defined here, so none stays alive across the epilogue of the
            // previous tile; steps past the end of the range are zero tiles that touch no memory
#pragma unroll
            for (int d = 0; d < PF; ++d) load_step(la[d], lb[d], AbS, BbS, rowS, colS, kB + d * BK, kE, d < full);
            la[0].store(As[0], tid);
            lb[0].store(Bs[0], tid);
            __syncthreads();
            for (int kt0 = 0; kt0 < nkS; kt0 += PF) {
#pragma unroll
                for (int u = 0; u < PF; ++u) {
                    const int kt = kt0 + u;
                    if (kt >= nkS) break;
                    const int cur = kt & 1;
                    if (kt + PF < nkS)
                        load_step(la[u], lb[u], AbS, BbS, rowS, colS, kB + (kt + PF) * BK, kE, kt + PF < full);
                    compute_step(As[cur], Bs[cur]);
                    if (kt + 1 < nkS) {
                        la[(u + 1) % PF].store(As[cur ^ 1], tid);
                        lb[(u + 1) % PF].store(Bs[cur ^ 1], tid);
                    }
                    __syncthreads();
                }
            }
            // the lane's output offsets are recomputed for every tile (the compiler would otherwise
            // keep them in registers across the K loop, which has none to spare)
            int laneE = lane;
            asm volatile("" : "+v"(laneE));
            if (ks0 == 0 && ks1 == nkT) {
                float *CbS = p.C + (long long)tcS.batch * p.strideC;
                write_tile_mfma32<false, FM, FN>(p, tcS, CbS, rowS + subM, colS + subN, laneE, acc32);
            } else {
                sk_store_part<BM, BN, FM, FN>(p, group, head, wave, laneE, acc32);
            }
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc32[i][j][e] = 0.f;
        });
        return;
    }

    pa.init(p.lda, row0, p.M, tid);
    pb.init(p.ldb, col0, p.N, tid);
    const int full = whole_steps(kBegin, kEnd);
#pragma unroll
    for (int d = 0; d < PF; ++d)
        if (d < nk) load_step(la[d], lb[d], Ab, Bb, row0, col0, kBegin + d * BK, kEnd, d < full);
    if (nk > 0) {
        la[0].store(As[0], tid);
        lb[0].store(Bs[0], tid);
    }
    __syncthreads();

    // K-step kt sits in LDS buffer kt & 1 and came through staging set kt % PF; while it is being
    // consumed, that set is refilled with step kt + PF and step kt + 1 moves from its set to LDS.
    for (int kt0 = 0; kt0 < nk; kt0 += PF) {
#pragma unroll
        for (int u = 0; u < PF; ++u) {
            const int kt = kt0 + u;
            if (kt >= nk) break;
            const int cur = kt & 1;
            if (kt + PF < nk) load_step(la[u], lb[u], Ab, Bb, row0, col0, kBegin + (kt + PF) * BK, kEnd, kt + PF < full);
            const float *as = As[cur], *bs = Bs[cur];
            compute_step(as, bs);
            if (kt + 1 < nk) {
                la[(u + 1) % PF].store(As[cur ^ 1], tid);
                lb[(u + 1) % PF].store(Bs[cur ^ 1], tid);
            }
            __syncthreads();
        }
    }

    // epilogue
    if constexpr (CORE == CORE_FMA) {
        write_tile<SPLIT>(p, tc, Cb, [&](auto emit) {
#pragma unroll
            for (int i = 0; i < P1; ++i)
#pragma unroll
                for (int j = 0; j < P2; ++j) emit(row0 + subM + i, col0 + subN + j, accF[i][j]);
        });
    } else if constexpr (KW > 1) {
        constexpr int CH = CORE == CORE_MFMA32 ? 4 : 1, FRG = CORE == CORE_MFMA32 ? 32 : 16;
        constexpr int UNITS = (NT / 64) * FM * FN * CH * 64;
        __shared__ floatx4 part[KW][UNITS];
        if constexpr (CORE == CORE_MFMA16) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) part[grp][((wave * FM + i) * FN + j) * 64 + lane] = acc16[i][j];
        } else {
            store_units32<FM, FN>(part[grp], wave, lane, acc32);
        }
        __syncthreads();
        store_sum_of_groups<SPLIT, FRG, CH, FM, FN, P1, P2, BN, NT, KW>(&part[0][0], p, tc, Cb, row0, col0);
    } else if constexpr (CORE == CORE_MFMA16) {
        write_tile_mfma16<SPLIT, FM, FN>(p, tc, Cb, row0 + subM, col0 + subN, lane, acc16);
    } else {
        write_tile_mfma32<SPLIT, FM, FN>(p, tc, Cb, row0 + subM, col0 + subN, lane, acc32);
    }
}

// Second kernel of the balanced persistent form: one single-wave work-group per left-over tile and
// wave tile (blockIdx.x = tile, blockIdx.y = wave of the first kernel's work-group).  A tile that
// one share covered whole was written by the first kernel and is skipped; for a divided tile the
// raw accumulator tiles of its shares are added in K order (ascending work-group, a fixed order:
// results are reproducible) and stored through the usual epilogue.  Lanes map to accumulator
// elements exactly as in gemm_f32_kernel.
template <int BM, int BN, int BK, int P1, int P2>
__global__ __launch_bounds__(64) void gemm_f32_sk_fixup_kernel(const GemmParams p) {
    constexpr int FM = P1 / 32, FN = P2 / 32;
    const long long groups = p.skGroups;
    const int nkT = (p.K + BK - 1) / BK;
    const long long units = (long long)p.skTailTiles * nkT;
    const long long t = blockIdx.x, u0 = t * nkT, u1 = u0 + nkT;
    // first work-group whose share reaches into this tile
    long long w = (u0 * groups) / units;
    while (w > 0 && sk_share_begin(w, units, groups) > u0) --w;
    while (sk_share_begin(w + 1, units, groups) <= u0) ++w;
    if (sk_share_begin(w, units, groups) <= u0 && sk_share_begin(w + 1, units, groups) >= u1) return;

    const int lane = (int)threadIdx.x, wave = (int)blockIdx.y;
    floatx16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // the parts are fetched four shares at a time (all loads of a batch are independent) and
    // added in share order
    constexpr int PB = 4;
    bool more = true;
    do {
        const floatx4 *part[PB];
        bool have[PB];
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            have[q] = false;
            part[q] = nullptr;
            while (more) {
                if (w >= groups) { more = false; break; }
                const long long b = sk_share_begin(w, units, groups), e = sk_share_begin(w + 1, units, groups);
                if (b >= u1) { more = false; break; }
                const long long cur = w++;
                if (e <= b) continue;                        // an empty share wrote nothing
                part[q] = reinterpret_cast<const floatx4 *>(p.ws) + (cur * 2 + (b / nkT == t ? 0 : 1)) * (BM * BN / 4) +
                          (long long)wave * (FM * FN * 4 * 64) + lane;
                have[q] = true;
                break;
            }
        }
        floatx4 v[PB][FM * FN * 4];
#pragma unroll
        for (int q = 0; q < PB; ++q)
            if (have[q]) {
#pragma unroll
                for (int f = 0; f < FM * FN * 4; ++f) v[q][f] = part[q][f * 64];
            }
#pragma unroll
        for (int q = 0; q < PB; ++q)
            if (have[q]) {
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
#pragma unroll
                            for (int x = 0; x < 4; ++x) acc[i][j][4 * c + x] += v[q][(i * FN + j) * 4 + c][x];
            }
    } while (more);
    const TileCoord tc = tile_of_logical(p, (unsigned)p.skRounds * (unsigned)groups + (unsigned)t);
    float *Cb = p.C + (long long)tc.batch * p.strideC;
    const int subM = (wave / (BN / P2)) * P1, subN = (wave % (BN / P2)) * P2;
    write_tile_mfma32<false, FM, FN>(p, tc, Cb, tc.tm * BM + subM, tc.tn * BN + subN, lane, acc);
}

}  // namespace ks
