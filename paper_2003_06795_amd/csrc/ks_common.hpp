// Shared device-side pieces of the tiled GEMM family (paper Section II): launch parameters,
// work-group -> tile mapping, and the alpha/beta epilogue.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ks {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// Four floats at an address that only the element type aligns: global memory takes sixteen-byte accesses
// at any element (the target's unaligned access mode), so this is one global_load_dwordx4 like the aligned form.
struct __attribute__((packed, aligned(4))) AnyFloatx4 {
    floatx4 v;
};
__device__ __forceinline__ floatx4 load_float4_any(const void *src) { return static_cast<const AnyFloatx4 *>(src)->v; }
// and eight 16-bit elements
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(2))) AnyUintx4 {
    uintx4 v;
};
__device__ __forceinline__ uintx4 load16_any(const uint16_t *src) {
    return reinterpret_cast<const AnyUintx4 *>(src)->v;
}
// and four, of an output kept in bf16
typedef unsigned int uintx2 __attribute__((ext_vector_type(2)));
struct __attribute__((packed, aligned(2))) AnyUintx2 {
    uintx2 v;
};

// n / d for n < 2^31, as a multiplication and a shift that the scalar unit does: there is no integer division, and what the
// compiler puts in its place, some 25 dependent instructions of the vector unit for each of the four that find a tile, was
// most of the time from the kernel's arguments to its first load.  1024 x 32x64x16 fp32 on 32 x 32 tiles 6.55 -> 5.86 us, 700 x
// 60x52x33 11.2 -> 10.3, 401408 x 64 x 27 39.0 -> 38.2; level from 20 us on where tiles have more than a few K-steps
// (480 x 1184 x 2592 TN 31.7 -> 31.6).
// m = ceil(2^(31 + s) / d) with 2^(s - 1) < d <= 2^s: m d exceeds 2^(31 + s) by less than 2^s, which n < 2^31 makes less than one
// part in d of a quotient's unit.
struct Divisor {
    unsigned mul, shift;
};
inline Divisor divisor_of(unsigned d) {
    const unsigned s = d > 1 ? 32 - (unsigned)__builtin_clz(d - 1) : 0;
    return Divisor{(unsigned)(((1ULL << (31 + s)) + d - 1) / d), 31 + s};
}
__host__ __device__ __forceinline__ unsigned divide(unsigned n, Divisor d) {
    return (unsigned)((unsigned long long)n * d.mul >> d.shift);
}

// (arguments lie in memory that no cache of the device holds at a launch; what a three-dimensional launch reads before its first
// loads stays in the first 144 bytes and in one group of loads: with perSplit at byte 188, or with C further back, which the compiler
// then fetched in a second group, every launch took 0.2 us more)
struct GemmParams {
    Divisor perSplit;                // K partitions (tile order, set_tile_order)
    const void *A;
    const void *B;
    float *C;
    float *ws;                       // split-K partial sums: [split][batch][M][N], dense
    const float *bias;               // N values added to every row of C after alpha / beta, or null
    long long lda, ldb, ldc;
    long long strideA, strideB, strideC;
    int M, N, K, batch;
    int tilesM, tilesN;
    int splitK, kChunk;              // K range of split s is [s*kChunk, min(K, (s+1)*kChunk))
    int grid3d;                      // 1: launched as (tilesN, tilesM, batch*splitK) work-groups
    int tilesPerWG;                  // consecutive logical tiles one work-group walks (members that
                                     // support it; 1 everywhere else and on 3-D launches)
    int bandRows;                    // tile rows per band of the one-dimensional tile order (8 unless the
                                     // member says otherwise)
    int out16;                       // 1: C holds bf16 (2-byte elements; ldc in elements); strideC is
                                     //    then 0 and the batch stride, in elements, is strideC16
    long long strideC16;
    float alpha, beta;
    // tile order: tiles of a unit, tiles of a band, rows of a band and of the last one
    Divisor perUnit, perBand, perRow, perLastRow;
    // balanced persistent form (fp32 members that have one; 0 everywhere else): the launch holds
    // skGroups work-groups; each computes skRounds whole tiles (logical tiles round * skGroups + its
    // own logical id) and then an equal share of the K-steps of the skTailTiles tiles that are left
    int skGroups, skRounds, skTailTiles;
    // a launch over part of the tiles (the split tail of a hybrid launch, see dispatch.hip): logical
    // ids 0 .. tileSpan * splitK - 1 stand for the tiles tileBase .. tileBase + tileSpan - 1 of the
    // one-dimensional order, partition-major, and partial sums go to the workspace as compact
    // bm x bn tiles [partition][tile - tileBase].  tileSpan == 0 everywhere else.
    int tileBase, tileSpan, bm, bn;
};
// from the tile counts, the partitions and the band height, once they are final (a three-dimensional launch reads its tile)
inline void set_tile_order(GemmParams &p) {
    if (p.grid3d) {
        if (p.splitK > 1) p.perSplit = divisor_of((unsigned)p.splitK);
        return;
    }
    p.perUnit = divisor_of(p.tileSpan ? (unsigned)p.tileSpan : (unsigned)p.tilesM * (unsigned)p.tilesN);
    p.perSplit = divisor_of((unsigned)p.splitK);
    p.perBand = divisor_of((unsigned)p.bandRows * (unsigned)p.tilesN);
    p.perRow = divisor_of((unsigned)p.bandRows);
    p.perLastRow = divisor_of((unsigned)((p.tilesM - 1) % p.bandRows + 1));
}

// What a launch of one batch item and no K partitions that reads its tile needs before its first loads, as three arguments in front
// of the others: the build has the compiler put the first fourteen dwords into scalar registers when a wave starts
// (-amdgpu-kernarg-preload-count), where all others come from memory that no cache holds at a launch.  Three vectors, because the
// runtime copies argument by argument (eleven scalars cost the host 0.15 us a call).  For the kernels of short calls, us, launches
// of a graph: fp32 73 x 57 x 232 NT (K-sliced) 3.09 -> 2.66, 359 x 69 x 24 NT (direct) 2.48 -> 2.18, 200 x 300 x 700 NT 5.05 -> 4.65, 37 x 1001 x 515
// NT 4.82 -> 4.75; bf16 128 x 128 x 2048 NT (K slices) 3.29 -> 3.21, 512 x 512 x 512 NT 3.14 -> 3.07; level to 1 % the other way elsewhere.
// Calls that wait for the host (128 x 128 x 128 fp32: kernel 3.1, call 4.1) show nothing of it.
typedef unsigned long long HotPointers __attribute__((ext_vector_type(2)));
typedef int HotInts __attribute__((ext_vector_type(4)));
#define KS_PARAMS const HotPointers hotAB, const HotInts hotSizes, const HotInts hotForm, const GemmParams rest
#define KS_ARGUMENTS(p)                                                                                                          \
    HotPointers{(unsigned long long)(uintptr_t)(p).A, (unsigned long long)(uintptr_t)(p).B},                                  \
        HotInts{(int)(p).lda, (int)(p).ldb, (p).M, (p).N}, HotInts{(p).K, (p).kChunk, (p).grid3d, (p).splitK}, (p)
#define KS_PARAMS_TOGETHER                                                                                                        \
    GemmParams p = rest;                                                                                                          \
    p.A = reinterpret_cast<const void *>((uintptr_t)hotAB.x); p.B = reinterpret_cast<const void *>((uintptr_t)hotAB.y);           \
    p.lda = hotSizes.x; p.ldb = hotSizes.y; p.M = hotSizes.z; p.N = hotSizes.w;                                                   \
    p.K = hotForm.x; p.kChunk = hotForm.y; p.grid3d = hotForm.z; p.splitK = hotForm.w

// origin of a batch item; the stride of the first one is not waited for
template <class T>
__device__ __forceinline__ T *batch_origin(T *base, int batch, long long stride) {
    if (batch != 0) {
        asm volatile("");                                    // (keeps the stride, and the wait for it, in here)
        base += batch * stride;
    }
    return base;
}

// K-steps [first, last) of the left-over tiles (flattened as tile * steps-per-tile + step) that
// work-group `w` of `groups` computes in the balanced persistent form; shares differ by at most one
__host__ __device__ inline long long sk_share_begin(long long w, long long units, long long groups) {
    return (w * units) / groups;
}

// bf16 <-> fp32 for an output kept in bf16: widening is exact, narrowing rounds to nearest even
// (NaN stays NaN)
__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
    return __builtin_bit_cast(float, (unsigned)b << 16);
}
__device__ __forceinline__ uint16_t float_to_bf16_bits(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}
// C[idx] = alpha * acc + beta * C[idx] + bias with C in bf16 (element index idx from the batch
// item's origin)
__device__ __forceinline__ void store_bf16_out(float *Cb, long long idx, float acc, float alpha, float beta,
                                               float biasv) {
    uint16_t *c = reinterpret_cast<uint16_t *>(Cb) + idx;
    float x = alpha * acc;
    if (beta != 0.0f) x = fmaf(beta, bf16_bits_to_float(*c), x);
    *c = float_to_bf16_bits(x + biasv);
}

// How the LDS-staged fp32 members (nt threads to a group of waves) fetch a K-step: one of three forms of the
// kernel.  STEPS reads whole K-steps without a test, sixteen bytes per lane at any element, and the step that
// holds the end of K in a second way; UNITS knows one way, a test per sixteen bytes, for extents that are
// multiples of four; ELEMENTS reads four bytes per lane and test.
enum { LOAD_STEPS = 0, LOAD_UNITS = 1, LOAD_ELEMENTS = 2 };
// threads that find nothing to fetch in a K-step of sixteen-byte units
constexpr bool f32_idle_threads(int rows, int bk, int nt) { return (rows * bk / 4) % nt != 0; }
// UNITS at any K.  The second way of STEPS is code that a short K-step does not amortise, and threads without a
// unit branch around every load: UNITS / STEPS over ten to forty K-steps, geometric means over the layouts, for
// idle threads 64 x 32 x 32 0.91, 32 x 64 x 32 0.90, 16 x 16 x 8 0.86, 32 x 32 x 16 0.85, 64 x 64 x 8 0.89, 16 x 128 x 16 0.88,
// 64 x 64 x 16 and x 32 with sixteen waves 0.93; one unit each: 32 x 32 x 32 with two K groups 0.97 (3928 x 24 x 1568 NN
// 13.4 -> 12.5 us), eight-wave 128 x 128 x 16 0.95; FMA 64 x 64 x 8 0.95.  Elsewhere 0.99 (64 x 64 x 16) to 1.11 (16 x 16 x 32).
constexpr bool f32_units_at_any_k(int core, int bm, int bn, int bk, int nt, int kw) {
    return core == 0 || f32_idle_threads(bm, bk, nt) || f32_idle_threads(bn, bk, nt) ||
           (bm * bk == 4 * nt && bn * bk == 4 * nt && (kw > 1 ? core == 1 : nt >= 512));
}
// No STEPS form: neither operand keeps the threads busy and the K-step is short.  ELEMENTS / STEPS on ragged
// operands over three to forty K-steps: 16 x 16 x 8 0.90, 32 x 32 x 16 0.92, 64 x 64 x 8 0.92, 64 x 64 x 16 0.91, FMA 32 x 32 x 8 0.88;
// the other members 1.0 to 1.5.
constexpr bool f32_never_steps(int bm, int bn, int bk, int nt) {
    return f32_idle_threads(bm, bk, nt) && f32_idle_threads(bn, bk, nt) && bk <= 16;
}
// K-steps up to which ragged operands take ELEMENTS in the members that have STEPS: where the step that holds
// the end of K is all there is (3136 x 256 x 3 NN on 64 x 64 x 16 3.8 -> 3.6 us, 196 x 512 x 27 on 32 x 32 x 32 3.05 -> 2.9), and
// where it is every second one for the members above that branch most (512 x 35x30x58 NT on 32 x 64 x 32 6.1 -> 5.7,
// 784 x 256 x 75 NN with two K groups 4.0 -> 3.7); behind by 5 - 20 % beyond, and by 8 - 13 % from the first with K groups
// of 64, whose steps are nearly all whole.
constexpr int f32_element_steps(int core, int bm, int bn, int bk, int nt, int kw) {
    return kw > 1 && bk >= 64                                                                        ? 0
           : f32_idle_threads(bm, bk, nt) || f32_idle_threads(bn, bk, nt) || (core == 1 && kw > 1) ? 2
                                                                                                     : 1;
}

// fp32 LDS-staged members that also exist in a form whose work-groups walk several tiles
// (GemmParams::tilesPerWG): 32x32 MFMA members (core 2) with large tiles of at least 128 columns
// (the 128 x 64 member measured slower in that form), wave tiles of at most 2048 entries (the form
// holds staging registers across the epilogue) and a single K group.
constexpr bool f32_multi_tile(int core, int bm, int bn, int p1, int p2, int kw) {
    return core == 2 && bm * bn >= 8192 && bn >= 128 && p1 * p2 <= 2048 && kw == 1;
}

// fp32 members with a form on the bf16 matrix pipe (gemm_f32_parts.hpp): the 128 x 128 x 32 tiles, and 64 x 64 x 16 ones unless
// K partitions of theirs have one group of waves each.
constexpr bool f32_parts_member(int core, int bm, int bn, int bk, int kw, bool split) {
    return core == 2 && ((bm == 128 && bn == 128 && bk == 32 && kw == 1) ||
                         (bm == 64 && bn == 64 && bk == 16 && (kw == 2 || (kw == 1 && !split))));
}
// It takes K ranges (of a work-group) from these on.  Time against the fp32 matrix pipe over drawn problems of 16 to 4096 in each
// dimension and im2col ones, all layouts, with and without scratch: 128 x 128 tiles 0.67 (98 problems; K of 49 to 64 0.89, 0.96 at
// most), 64 x 64 0.77 (101; 49 to 64 0.94, four of 40 over 1.02, and up to 48 half of them slower by up to 1.10), two K groups 0.87
// (101; ranges of 360 to 420 0.905, five of 40 over 1.02, 1.055 at most; below 360 half slower, up to 1.15, 0.95 in all: a few
// steps to a slice and one work-group to a compute unit wait for memory, which the fp32 form has four steps in flight for).
constexpr int f32_parts_least_k(int kw) { return kw == 2 ? 360 : 49; }
// In that form an unsplit 64 x 64 x 16 member computes 2 x 2 tiles per work-group, on the 128 x 128 tile of eight waves, where a
// work-group's sum of splitting and LDS traffic is half as long per product: the bits are the same.  Two of them fill a unit, so
// 512 make a round; the line lies where the rounds, in units of products, are not over 1.15 of those of 256 small tiles (an even
// share to a unit).  112 of 700 drawn problems of the unsplit member, 0.886 of the time, worst 1.05 (K from 128 on 0.85, up to
// 80 0.94 with one in ten over 1.03): 50176 x 95 x 2757 NN 289 -> 214 us.  With the line at 1.25 155 at 0.90, eight over 1.03.
constexpr bool f32_parts_square(int64_t tiles64, int64_t tiles128, int64_t K) {
    return K >= 80 && 160 * ((tiles128 + 511) / 512) <= 23 * ((tiles64 + 255) / 256);
}

// 16-bit members whose direct-to-LDS path runs in the form with two groups of waves alternating
// between memory and MFMA slots: the eight-wave 256 x 256 x 64 members (128 x 64 of output per wave)
// with either fragment shape, and the eight-wave 128 x 128 x 128 members on 16x16x32 fragments
// (64 x 32 of output per wave).
constexpr bool bf16_two_groups(int f, int bm, int bn, int bk, int wm, int wn, int stages) {
    return ((f == 32 || f == 16) && bm == 256 && bn == 256 && bk == 64 && wm == 128 && wn == 64 && stages == 2) ||
           (f == 16 && bm == 128 && bn == 128 && bk == 128 && wm == 64 && wn == 32 && stages == 2);
}

// launch shape that tile_of_block expects
inline dim3 launch_grid(const GemmParams &p, int grid) {
    return p.grid3d ? dim3((unsigned)p.tilesN, (unsigned)p.tilesM, (unsigned)(p.batch * p.splitK))
                    : dim3((unsigned)grid);
}

struct TileCoord {
    int batch, split, tm, tn;
};

// MI355X has 8 XCDs with private L2s and hands consecutive work-group ids to them round-robin.
// Renumber so that each XCD owns one contiguous run of logical tile ids, then walk tiles in
// bands of a few tile-rows (8 by default; a tunable axis of the 16-bit family), column-major inside
// a band, so the tiles resident on one XCD form a compact block that shares A row-panels and B
// column-panels in that XCD's L2.
// Small grids (where a handful of integer divisions is a visible part of a 3 us kernel and L2
// locality is not at stake) are launched three-dimensional instead and read their tile directly.
__device__ __forceinline__ unsigned logical_of_block() {
    const unsigned total = gridDim.x, id = blockIdx.x;
    const unsigned q = total >> 3, r = total & 7u, x = id & 7u;
    return x * q + (x < r ? x : r) + (id >> 3);
}

// tile with logical id `logical` of a one-dimensional launch: units (batch item, K partition) in
// order, inside a unit bands of p.bandRows tile-rows walked column-major
__device__ __forceinline__ TileCoord tile_of_logical(const GemmParams &p, unsigned logical) {
    const unsigned per = p.tileSpan ? (unsigned)p.tileSpan : (unsigned)p.tilesM * (unsigned)p.tilesN;
    const unsigned unit = divide(logical, p.perUnit), t = logical - unit * per + (unsigned)p.tileBase;
    TileCoord c;
    c.batch = (int)divide(unit, p.perSplit);
    c.split = (int)(unit - (unsigned)c.batch * (unsigned)p.splitK);
    const unsigned h = (unsigned)p.bandRows;
    const unsigned band = h * (unsigned)p.tilesN;
    const unsigned g = divide(t, p.perBand), in = t - g * band;
    const unsigned first = g * h;
    const bool last = (unsigned)p.tilesM - first < h;
    const unsigned rows = last ? (unsigned)p.tilesM - first : h;
    c.tn = (int)divide(in, Divisor{last ? p.perLastRow.mul : p.perRow.mul, last ? p.perLastRow.shift : p.perRow.shift});
    c.tm = (int)(first + (in - (unsigned)c.tn * rows));
    return c;
}

// inverse of the tile walk above: position of tile (tm, tn) in the one-dimensional order of a unit
__device__ __forceinline__ unsigned logical_of_tile(const GemmParams &p, int tm, int tn) {
    const unsigned h = (unsigned)p.bandRows;
    const unsigned g = divide((unsigned)tm, p.perRow), first = g * h;
    const unsigned rows = ((unsigned)p.tilesM - first) < h ? ((unsigned)p.tilesM - first) : h;
    return g * h * (unsigned)p.tilesN + (unsigned)tn * rows + ((unsigned)tm - first);
}

// Where a split-K instantiation puts its partial sums and with which row length: the dense
// [partition][batch][M][N] array, or, in a launch over part of the tiles, the compact tile
// [partition][tile - tileBase] (the returned base is shifted so that base + row * ld + col with
// the absolute row and column lands inside that tile).
__device__ __forceinline__ float *partial_base(const GemmParams &p, const TileCoord &tc, long long &ld) {
    if (p.tileSpan) {
        ld = p.bn;
        const long long tileElems = (long long)p.bm * p.bn;
        const long long rel = (long long)logical_of_tile(p, tc.tm, tc.tn) - p.tileBase;
        return p.ws + ((long long)tc.split * p.tileSpan + rel) * tileElems -
               ((long long)tc.tm * p.bm * p.bn + (long long)tc.tn * p.bn);
    }
    ld = p.N;
    return p.ws + ((long long)tc.split * p.batch + tc.batch) * (long long)p.M * p.N;
}

__device__ __forceinline__ TileCoord tile_of_block(const GemmParams &p) {
    if (p.grid3d) {
        TileCoord c;
        c.tn = (int)blockIdx.x;
        c.tm = (int)blockIdx.y;
        const unsigned unit = blockIdx.z;
        if (p.splitK == 1) {
            c.batch = (int)unit; c.split = 0;
        } else {
            c.batch = (int)divide(unit, p.perSplit);
            c.split = (int)(unit - (unsigned)c.batch * (unsigned)p.splitK);
        }
        return c;
    }
    return tile_of_logical(p, logical_of_block());
}

// Epilogue.  `visit(f)` calls f(row, col, acc) for every accumulator element this lane owns
// (tile-relative to the matrix, i.e. absolute row / col).  The three output modes are separated
// outside the element loops so the per-element code is a bounds test and one store:
//   SPLIT (a split-K instantiation): raw partial sum to this split's slice of the workspace;
//   beta == 0: C = alpha * acc (C is never read);
//   otherwise: C = alpha * acc + beta * C;
//   with a bias vector, bias[col] is added last (a split-K instantiation leaves that to the
//   reduction pass).
template <bool SPLIT, class Visit>
__device__ __forceinline__ void write_tile(const GemmParams &p, const TileCoord &tc, float *Cb,
                                           Visit visit) {
    const int M = p.M, N = p.N;
    if constexpr (SPLIT) {
        long long wld;
        float *w = partial_base(p, tc, wld);
        visit([&](int row, int col, float acc) {
            if (row < M && col < N) w[(long long)row * wld + col] = acc;
        });
    } else if (p.out16) {
        const float alpha = p.alpha, beta = p.beta;
        const float *bias = p.bias;
        const long long ldc = p.ldc;
        visit([&](int row, int col, float acc) {
            if (row < M && col < N)
                store_bf16_out(Cb, (long long)tc.batch * p.strideC16 + (long long)row * ldc + col, acc, alpha,
                               beta, bias ? bias[col] : 0.0f);
        });
    } else if (p.bias != nullptr) {
        const float alpha = p.alpha, beta = p.beta;
        const float *bias = p.bias;
        const long long ldc = p.ldc;
        visit([&](int row, int col, float acc) {
            if (row < M && col < N) {
                float *c = Cb + (long long)row * ldc + col;
                float v = alpha * acc;
                if (beta != 0.0f) v = fmaf(beta, *c, v);
                *c = v + bias[col];
            }
        });
    } else if (p.beta == 0.0f) {
        const float alpha = p.alpha;
        const long long ldc = p.ldc;
        visit([&](int row, int col, float acc) {
            if (row < M && col < N) Cb[(long long)row * ldc + col] = alpha * acc;
        });
    } else {
        const float alpha = p.alpha, beta = p.beta;
        const long long ldc = p.ldc;
        visit([&](int row, int col, float acc) {
            if (row < M && col < N) {
                float *c = Cb + (long long)row * ldc + col;
                *c = fmaf(beta, *c, alpha * acc);
            }
        });
    }
}

// Where an accumulator tile goes: the matrix C (alpha, beta applied) or, in a split-K
// instantiation, this partition's slice of the workspace (raw partial sums, dense rows of N).
struct OutTarget {
    float *base;
    const float *bias;               // added after alpha / beta; null in split-K instantiations
    long long ld;
    float alpha, beta;
    int M, N;
    int out16;                       // C is bf16 (never set in split-K instantiations)
    long long off16;                 // element offset of the batch item in a bf16 C
};

template <bool SPLIT>
__device__ __forceinline__ OutTarget out_target(const GemmParams &p, const TileCoord &tc, float *Cb) {
    OutTarget o;
    o.M = p.M; o.N = p.N;
    if constexpr (SPLIT) {
        o.base = partial_base(p, tc, o.ld);
        o.alpha = 1.0f; o.beta = 0.0f; o.bias = nullptr; o.out16 = 0; o.off16 = 0;
    } else {
        o.base = Cb; o.ld = p.ldc; o.alpha = p.alpha; o.beta = p.beta; o.bias = p.bias; o.out16 = p.out16;
        o.off16 = (long long)tc.batch * p.strideC16;
    }
    return o;
}

// One lane's share of an MFMA fragment: NE values in one column `col`, at rows r0 + rowOff(e).
// `full` (the same for every lane of the wave) says the whole fragment lies inside the matrix:
// then there is no per-element test, and with beta != 0 all the old values are fetched before the
// first one is needed.  Edge fragments test every element.
template <bool SPLIT, int NE, class RowOff>
__device__ __forceinline__ void store_lane_column(const OutTarget &o, int r0, int col, bool full,
                                                  const float (&v)[NE], RowOff rowOff) {
    if (!SPLIT && o.out16) {
        // bf16 output: one form for interior and edge fragments
        if (col < o.N) {
            const float bv = o.bias ? o.bias[col] : 0.0f;
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (r0 + rowOff(e) < o.M)
                    store_bf16_out(o.base, o.off16 + (long long)(r0 + rowOff(e)) * o.ld + col, v[e], o.alpha,
                                   o.beta, bv);
        }
        return;
    }
    float *ptr = o.base + (long long)r0 * o.ld + col;
    if (!SPLIT && o.bias != nullptr) {
        // bias form: the lane's column is fixed, so one bias value serves all its elements
        if (col < o.N) {
            const float bv = o.bias[col];
            float old[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e)
                old[e] = (o.beta != 0.0f && r0 + rowOff(e) < o.M) ? ptr[(long long)rowOff(e) * o.ld] : 0.0f;
#pragma unroll
            for (int e = 0; e < NE; ++e)
                if (r0 + rowOff(e) < o.M) {
                    float x = o.alpha * v[e];
                    if (o.beta != 0.0f) x = fmaf(o.beta, old[e], x);
                    ptr[(long long)rowOff(e) * o.ld] = x + bv;
                }
        }
    } else if (full) {
        if (SPLIT) {
#pragma unroll
            for (int e = 0; e < NE; ++e) ptr[(long long)rowOff(e) * o.ld] = v[e];
        } else if (o.beta == 0.0f) {
#pragma unroll
            for (int e = 0; e < NE; ++e) ptr[(long long)rowOff(e) * o.ld] = o.alpha * v[e];
        } else {
            float old[NE];
#pragma unroll
            for (int e = 0; e < NE; ++e) old[e] = ptr[(long long)rowOff(e) * o.ld];
#pragma unroll
            for (int e = 0; e < NE; ++e) ptr[(long long)rowOff(e) * o.ld] = fmaf(o.beta, old[e], o.alpha * v[e]);
        }
    } else if (col < o.N) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            if (r0 + rowOff(e) < o.M) {
                float *c = ptr + (long long)rowOff(e) * o.ld;
                if (SPLIT) *c = v[e];
                else if (o.beta == 0.0f) *c = o.alpha * v[e];
                else *c = fmaf(o.beta, *c, o.alpha * v[e]);
            }
        }
    }
}

// accumulator register e of lane l of a 16x16 MFMA fragment holds C[4*(l/16) + e][l%16]
template <bool SPLIT, int FM, int FN, class Acc>
__device__ __forceinline__ void write_tile_mfma16(const GemmParams &p, const TileCoord &tc, float *Cb,
                                                  int rowBase, int colBase, int lane, const Acc &acc) {
    const OutTarget o = out_target<SPLIT>(p, tc, Cb);
    const int rb = __builtin_amdgcn_readfirstlane(rowBase), cb = __builtin_amdgcn_readfirstlane(colBase);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const bool full = rb + i * 16 + 16 <= o.M && cb + j * 16 + 16 <= o.N;
            const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
            store_lane_column<SPLIT, 4>(o, rb + i * 16 + 4 * (lane >> 4), cb + j * 16 + (lane & 15), full, v,
                                        [](int e) { return e; });
        }
}

// Four consecutive entries of a row of C, columns col .. col + 3: what a lane holds of a 16x16 fragment that is computed with the
// operands exchanged, B op(A): register e of lane l is then C[l%16][4*(l/16) + e], a neighbour in a row and not in a column, and
// the entries are one access of sixteen bytes (eight in bf16) where they were four of four (two).  For the kernels whose epilogue
// counts, those in two groups of waves (gemm_bf16_pp.hpp); members of a few microseconds lost 0.1 - 0.2 us by the longer code.
// `full` as above.  old_entries() is apart from store_entries() so that old values can be requested before the first store.
__device__ __forceinline__ floatx4 old_entries(const OutTarget &o, int row, int col, bool full) {
    floatx4 old = {0.f, 0.f, 0.f, 0.f};
    const long long at = (long long)row * o.ld + col;
    if (o.out16) {
        const uint16_t *c = reinterpret_cast<const uint16_t *>(o.base) + o.off16 + at;
        if (full) {
            const uintx2 u = reinterpret_cast<const AnyUintx2 *>(c)->v;
#pragma unroll
            for (int e = 0; e < 4; ++e) old[e] = bf16_bits_to_float((uint16_t)(u[e >> 1] >> (16 * (e & 1))));
        } else if (row < o.M) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < o.N) old[e] = bf16_bits_to_float(c[e]);
        }
    } else if (full) {
        old = load_float4_any(o.base + at);
    } else if (row < o.M) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < o.N) old[e] = o.base[at + e];
    }
    return old;
}
template <bool SPLIT>
__device__ __forceinline__ void store_entries(const OutTarget &o, int row, int col, bool full, floatx4 v, floatx4 old) {
    const long long at = (long long)row * o.ld + col;
    if constexpr (!SPLIT) {
        v = o.alpha * v;
        if (o.beta != 0.0f) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaf(o.beta, old[e], v[e]);
        }
        if (o.bias != nullptr) {
            if (full) v += load_float4_any(o.bias + col);
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < o.N) v[e] += o.bias[col + e];
        }
        if (o.out16) {
            uint16_t *c = reinterpret_cast<uint16_t *>(o.base) + o.off16 + at;
            const unsigned h[4] = {float_to_bf16_bits(v[0]), float_to_bf16_bits(v[1]), float_to_bf16_bits(v[2]),
                                   float_to_bf16_bits(v[3])};
            if (full) {
                reinterpret_cast<AnyUintx2 *>(c)->v = uintx2{h[0] | h[1] << 16, h[2] | h[3] << 16};
            } else if (row < o.M) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < o.N) c[e] = (uint16_t)h[e];
            }
            return;
        }
    }
    if (full) {
        reinterpret_cast<AnyFloatx4 *>(o.base + at)->v = v;
    } else if (row < o.M) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < o.N) o.base[at + e] = v[e];
    }
}

// accumulator register e of lane l of a 32x32 MFMA fragment holds C[8*(e/4) + 4*(l/32) + e%4][l%32]
template <bool SPLIT, int FM, int FN, class Acc>
__device__ __forceinline__ void write_tile_mfma32(const GemmParams &p, const TileCoord &tc, float *Cb,
                                                  int rowBase, int colBase, int lane, const Acc &acc) {
    const OutTarget o = out_target<SPLIT>(p, tc, Cb);
    const int rb = __builtin_amdgcn_readfirstlane(rowBase), cb = __builtin_amdgcn_readfirstlane(colBase);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const bool full = rb + i * 32 + 32 <= o.M && cb + j * 32 + 32 <= o.N;
            float v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = acc[i][j][e];
            store_lane_column<SPLIT, 16>(o, rb + i * 32 + 4 * (lane >> 5), cb + j * 32 + (lane & 31), full, v,
                                         [](int e) { return 8 * (e >> 2) + (e & 3); });
        }
}

// The same fragment layout written in four chunks of four rows with the scheduler kept from
// merging them: fewer addresses and old values alive at once, for kernels that hold other
// registers (the next tile's operands) across the epilogue.
template <bool SPLIT, int FM, int FN, class Acc>
__device__ __forceinline__ void write_tile_mfma32_lean(const GemmParams &p, const TileCoord &tc, float *Cb,
                                                       int rowBase, int colBase, int lane, const Acc &acc) {
    const OutTarget o = out_target<SPLIT>(p, tc, Cb);
    const int rb = __builtin_amdgcn_readfirstlane(rowBase), cb = __builtin_amdgcn_readfirstlane(colBase);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            const bool full = rb + i * 32 + 32 <= o.M && cb + j * 32 + 32 <= o.N;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float v[4] = {acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
                store_lane_column<SPLIT, 4>(o, rb + i * 32 + 8 * c + 4 * (lane >> 5), cb + j * 32 + (lane & 31), full, v,
                                            [](int e) { return e; });
                __builtin_amdgcn_sched_barrier(0);
            }
        }
}

}  // namespace ks
