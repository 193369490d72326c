// Host side of the C ABI: argument validation, registry, launch geometry, timing helper.
// Every compute step runs in the HIP kernels of this library; there is no CPU fallback.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "../../include/ks_gemm.h"
#include "registry.hpp"
#include "slices.hpp"

#ifndef KS_GRID3D_MAX
#define KS_GRID3D_MAX 2048      // work-groups up to which the grid is launched three-dimensional
#endif
#ifndef KS_GRID3D_BYTES
#define KS_GRID3D_BYTES (4 << 20)   // ... and bytes of A and B together
#endif

namespace ks {

// selector.cpp
int select_member(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int transA, int transB, bool scratch);
bool custom_tree(int dtype);
bool split_decides(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch);

#define KS_DECL(n)                              \
    void register_f32_shard_##n(LaunchFn *);    \
    void register_bf16_shard_##n(LaunchFn *);   \
    void register_bf16_dma_shard_##n(LaunchFn *);
KS_DECL(0) KS_DECL(1) KS_DECL(2) KS_DECL(3) KS_DECL(4) KS_DECL(5) KS_DECL(6) KS_DECL(7)
KS_DECL(8) KS_DECL(9) KS_DECL(10) KS_DECL(11) KS_DECL(12) KS_DECL(13) KS_DECL(14) KS_DECL(15)
#undef KS_DECL

namespace {

constexpr int threads_of(int core, int bm, int bn, int p1, int p2) {
    return core == KS_CORE_FMA ? (bm / p1) * (bn / p2) : core == KS_CORE_KSLICE ? 64 * p1 * (bm / p2) * (bn / p2) : 64 * (bm / p1) * (bn / p2);
}

constexpr int KS_CORE_OF_FMA = KS_CORE_FMA, KS_CORE_OF_MFMA16 = KS_CORE_MFMA16,
              KS_CORE_OF_MFMA32 = KS_CORE_MFMA32, KS_CORE_OF_DIRECT = KS_CORE_DIRECT,
              KS_CORE_OF_KSLICE = KS_CORE_KSLICE;

const InstanceDesc kF32[kNumF32] = {
// kw: K groups inside the work-group (K-sliced members: waves along K); LDS-staged members with
// K groups also hold the float4 units through which the groups' accumulators are added
#define KS_F32_INSTANCE_KW(id, CORE, BM, BN, BK, P1, P2, SPLITK, KW)                                     \
    {id, KS_CORE_OF_##CORE, BM, BN, BK, P1, P2, threads_of(KS_CORE_OF_##CORE, BM, BN, P1, P2) * (KW), SPLITK, \
     KS_CORE_OF_##CORE == KS_CORE_DIRECT   ? 0                                                          \
     : KS_CORE_OF_##CORE == KS_CORE_KSLICE ? P1 * BM * BN * 4                                           \
                                           : (KW) * 2 * BK * ((BM + (BK < 16 ? 64 / BK : 4)) + (BN + (BK < 16 ? 64 / BK : 4))) * 4 + \
                                                 ((KW) > 1 ? (KW) * BM * BN * 4 : 0),                     \
     KS_CORE_OF_##CORE == KS_CORE_KSLICE ? P1 : (KW)},
#define KS_F32_INSTANCE(id, CORE, BM, BN, BK, P1, P2, SPLITK) KS_F32_INSTANCE_KW(id, CORE, BM, BN, BK, P1, P2, SPLITK, 1)
#define KS_F32_INSTANCE_SK(id, CORE, BM, BN, BK, P1, P2, PERCU)                                          \
    {id, KS_CORE_OF_##CORE, BM, BN, BK, P1, P2, threads_of(KS_CORE_OF_##CORE, BM, BN, P1, P2), 1,         \
     2 * BK * ((BM + (BK < 16 ? 64 / BK : 4)) + (BN + (BK < 16 ? 64 / BK : 4))) * 4, 1, 8, PERCU},
#include "instances.def"
#undef KS_F32_INSTANCE
#undef KS_F32_INSTANCE_KW
#undef KS_F32_INSTANCE_SK
};

const InstanceDesc kBf16[kNumBf16] = {
#define KS_BF16_INSTANCE_BAND(id, F, BM, BN, BK, WM, WN, STAGES, SPLITK, BAND)                \
    {id, (F) == 16 ? KS_CORE_MFMA16 : KS_CORE_MFMA32, BM, BN, BK, WM, WN, 64 * (BM / WM) * (BN / WN), \
     SPLITK, STAGES * BK * (BM + BN) * 2, 1, BAND},
#define KS_BF16_INSTANCE(id, F, BM, BN, BK, WM, WN, STAGES, SPLITK) \
    KS_BF16_INSTANCE_BAND(id, F, BM, BN, BK, WM, WN, STAGES, SPLITK, 8)
#include "instances.def"
#undef KS_BF16_INSTANCE
#undef KS_BF16_INSTANCE_BAND
};

// granularity of K on the direct-to-LDS path: a member of K-step 128 takes half a step at the end
constexpr int64_t dma_k_step(const InstanceDesc &d) { return d.bk == 128 ? 64 : d.bk; }

LaunchFn g_f32[kNumF32];
LaunchFn g_bf16[kNumBf16];
LaunchFn g_bf16_dma[kNumBf16];
std::once_flag g_once;

void init_tables() {
    register_f32_shard_0(g_f32); register_f32_shard_1(g_f32); register_f32_shard_2(g_f32);
    register_f32_shard_3(g_f32); register_f32_shard_4(g_f32); register_f32_shard_5(g_f32);
    register_f32_shard_6(g_f32); register_f32_shard_7(g_f32); register_f32_shard_8(g_f32);
    register_f32_shard_9(g_f32); register_f32_shard_10(g_f32); register_f32_shard_11(g_f32);
    register_f32_shard_12(g_f32); register_f32_shard_13(g_f32); register_f32_shard_14(g_f32);
    register_f32_shard_15(g_f32);
    register_bf16_shard_0(g_bf16); register_bf16_shard_1(g_bf16); register_bf16_shard_2(g_bf16);
    register_bf16_shard_3(g_bf16); register_bf16_shard_4(g_bf16); register_bf16_shard_5(g_bf16);
    register_bf16_shard_6(g_bf16); register_bf16_shard_7(g_bf16); register_bf16_shard_8(g_bf16);
    register_bf16_shard_9(g_bf16); register_bf16_shard_10(g_bf16); register_bf16_shard_11(g_bf16);
    register_bf16_shard_12(g_bf16); register_bf16_shard_13(g_bf16); register_bf16_shard_14(g_bf16);
    register_bf16_shard_15(g_bf16);
    register_bf16_dma_shard_0(g_bf16_dma); register_bf16_dma_shard_1(g_bf16_dma);
    register_bf16_dma_shard_2(g_bf16_dma); register_bf16_dma_shard_3(g_bf16_dma);
    register_bf16_dma_shard_4(g_bf16_dma); register_bf16_dma_shard_5(g_bf16_dma);
    register_bf16_dma_shard_6(g_bf16_dma); register_bf16_dma_shard_7(g_bf16_dma);
    register_bf16_dma_shard_8(g_bf16_dma); register_bf16_dma_shard_9(g_bf16_dma);
    register_bf16_dma_shard_10(g_bf16_dma); register_bf16_dma_shard_11(g_bf16_dma);
    register_bf16_dma_shard_12(g_bf16_dma); register_bf16_dma_shard_13(g_bf16_dma);
    register_bf16_dma_shard_14(g_bf16_dma); register_bf16_dma_shard_15(g_bf16_dma);
}

int g_forceGeneric = 0;
int g_tilesPerWG = 0;        // 0: chosen per call (multi_tiles); n >= 1: forced
int g_skPerCU = 0;           // 0: the member's own count of work-groups per compute unit; n >= 1: forced
int g_tailSplit = -1;        // -1: chosen per call (tail_split); 0: never; n >= 2: forced where it can run
int g_operandCopies = -1;    // -1: chosen per call (copies_pay); 0: never; 1: wherever they can be made
int g_splitForced = 0;       // 0: per-call split members take auto_split's count; n >= 1: forced (at least two K-steps each)
void *g_ws = nullptr;
size_t g_wsBytes = 0;

// K partitions for an instance whose split is chosen per call.  Work-groups run in rounds of
// `slots` (256 compute units times the work-groups that fit one); a work-group costs its K-steps
// plus a fixed prologue/epilogue, and splitting adds the reduction pass.  The cheapest count wins
// (the smaller one on ties); never more than 64 (fp32) or 256 (16-bit), never more than fills one
// round (16-bit) or four (fp32), and at least two K-steps per partition.
//   fp32 members: twelve waves per compute unit, cost in K-steps as measured on the tuning set.
//   16-bit members: their LDS stages (up to 144 KB) limit a compute unit to one to four
//   work-groups, and a partition's tile of partial sums (written, then read by the reduction
//   pass) is charged in units of one K-step's operand traffic, 4 BM BN / ((BM + BN) BK).
int64_t split_slots(const InstanceDesc *d, bool f32) {
    const int64_t waves = d->threads / 64;
    int64_t perCU = 12 / waves > 0 ? 12 / waves : 1;
    if (!f32) {
        const int64_t byLds = d->ldsBytes > 0 ? (160 * 1024) / d->ldsBytes : perCU;
        perCU = byLds < perCU ? (byLds > 0 ? byLds : 1) : perCU;
    }
    return 256 * perCU;
}

int64_t auto_split_max(const InstanceDesc *d, int64_t tiles, bool f32) {
    const int64_t slots = split_slots(d, f32);
    int64_t s = (slots + tiles - 1) / (tiles > 0 ? tiles : 1);
    // fp32: up to four rounds of partitions.  A count that overfills one round can still end
    // sooner, e.g. 152 tiles in 5 partitions are three rounds of a fifth of K where unsplit tiles
    // are one round of all of it; the cost estimate below matched the measured order of the counts
    // on every shape tried.
    if (f32 && tiles > 0 && 4 * slots / tiles > s) s = 4 * slots / tiles;
    const int64_t cap = f32 ? 64 : 256;
    return s < 1 ? 1 : (s > cap ? cap : s);
}

int64_t auto_split(const InstanceDesc *d, int64_t tiles, int64_t kTiles, bool f32) {
    const int64_t slots = split_slots(d, f32);
    const int64_t partial = f32 ? 0 : (4LL * d->bm * d->bn) / ((int64_t)(d->bm + d->bn) * d->bk);
    int64_t best = 1, bestCost = -1;
    const int64_t smax = auto_split_max(d, tiles, f32);
    // kTiles counts the steps of the work-group.  The K groups of an LDS-staged member share the
    // compute unit's matrix pipe, so one of its steps lasts as many K-steps as it has groups; the
    // waves of a K-sliced member wait on memory side by side and a step lasts one.
    const int64_t stepCost = d->core != KS_CORE_KSLICE && d->kw > 1 ? d->kw : 1;
    for (int64_t s = 1; s <= smax && (s == 1 || 2 * s <= kTiles); ++s) {
        const int64_t rounds = (tiles * s + slots - 1) / slots;
        const int64_t cost = rounds * (stepCost * ((kTiles + s - 1) / s) + 6 + (s > 1 ? partial : 0)) + (s > 1 ? 10 : 0);
        if (bestCost < 0 || cost < bestCost) { bestCost = cost; best = s; }
    }
    return best;
}

// K partitions for the last, partly filled round of work-groups of a 16-bit member whose split is
// chosen per call (0 = launch every tile whole).  With `slots` work-groups resident at once, T
// tiles take ceil(T / slots) rounds although the last one may hold only a few tiles; cutting the
// K range of just those left-over tiles into s = slots / left-over partitions fills that round
// with work-groups that are s times shorter.  Same cost units as auto_split; the partitioned round
// also pays its tiles of partial sums and a third launch.  Only with at least one whole round
// before it (otherwise auto_split decides), and only when it saves 3 % of the call.
bool tail_split_member(const InstanceDesc *d) {
    // members whose LDS stages leave room for one work-group per compute unit: their round is 256
    // work-groups for certain (smaller members share a unit and suffer less from a short last round)
    return d->splitK == 0 && d->ldsBytes > 0 && (160 * 1024) / d->ldsBytes == 1;
}
// scratch of the largest partitioning tail_split can choose for this many tiles (0: no hybrid launch)
size_t tail_split_bytes(const InstanceDesc *d, int64_t tiles) {
    if (!tail_split_member(d)) return 0;
    const int64_t slots = split_slots(d, false);
    const int64_t tail = tiles % slots;
    if (tiles < slots || tail == 0) return 0;
    int64_t s = slots / tail;
    if (s > 16) s = 16;
    return s >= 2 ? (size_t)s * (size_t)tail * (size_t)d->bm * (size_t)d->bn * sizeof(float) : 0;
}
int64_t tail_split(const InstanceDesc *d, int64_t tiles, int64_t kTiles) {
    if (!tail_split_member(d)) return 0;
    const int64_t slots = split_slots(d, false);
    const int64_t rounds = tiles / slots, tail = tiles % slots;
    if (rounds == 0 || tail == 0) return 0;
    int64_t s = slots / tail;
    if (s > 16) s = 16;
    if (2 * s > kTiles) s = kTiles / 2;
    if (g_tailSplit >= 2) return s >= 2 ? (s < g_tailSplit ? s : g_tailSplit) : 0;
    if (s < 2) return 0;
    const int64_t partial = (4LL * d->bm * d->bn) / ((int64_t)(d->bm + d->bn) * d->bk);
    const int64_t plain = (rounds + 1) * (kTiles + 6);
    const int64_t hybrid = rounds * (kTiles + 6) + (kTiles + s - 1) / s + 6 + partial + 14;
    return 100 * hybrid <= 97 * plain ? s : 0;
}

// Tiles one work-group of a multi-tile fp32 member walks.  Walking T tiles takes the work-group
// launch, the pipeline fill and part of the wait behind the previous tile's stores out of T - 1 of
// T tiles, but leaves T times fewer work-groups to balance over the compute units, and the
// flattened loop itself is about 5 % slower per K-step.  Measured on outputs of 0.2 - 3.3 GB with
// T = 4 .. 8: 7 - 25 % faster when a tile has one K-step, 0 - 7 % with two, 5 % slower from four
// on; slower as soon as the launch has fewer than about ten rounds of work-groups.  Hence: only
// for tiles of at most two K-steps and at least 32 rounds of single-tile work-groups, and then so
// that 8 rounds remain (at most 8 tiles).
int multi_tiles(const InstanceDesc *d, int64_t tiles, int64_t K) {
    const int64_t waves = d->threads / 64;
    const int64_t slots = 256 * (12 / waves > 0 ? 12 / waves : 1);
    const int64_t rounds = tiles / slots;
    if (K > 2 * d->bk || rounds < 32) return 1;
    return (int)(rounds / 8 < 8 ? rounds / 8 : 8);
}

// Balanced persistent form: work-groups of the launch, and the scratch its divided tiles need (two
// raw accumulator tiles per work-group: the head and the tail of its share of the left-over tiles).
int64_t sk_groups(const InstanceDesc *d) { return 256LL * (g_skPerCU > 0 ? g_skPerCU : d->sk); }
size_t sk_workspace_bytes(const InstanceDesc *d) {
    return (size_t)sk_groups(d) * 2 * (size_t)d->bm * (size_t)d->bn * sizeof(float);
}

const InstanceDesc *desc_of(int dtype, int id) {
    if (dtype == KS_F32) return (id >= 0 && id < kNumF32) ? &kF32[id] : nullptr;
    if (dtype == KS_BF16 || dtype == KS_F16) return (id >= 0 && id < kNumBf16) ? &kBf16[id] : nullptr;
    return nullptr;
}

// C = beta * C (+ bias) for K == 0 (C is not read when beta == 0)
__global__ void scale_c_kernel(float *C, long long ldc, long long strideC, int M, int N, int batch,
                               float beta, const float *bias, int out16) {
    const long long total = (long long)batch * M * N;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
         i += (long long)gridDim.x * blockDim.x) {
        const long long b = i / ((long long)M * N), r = i - b * (long long)M * N;
        if (out16) {
            store_bf16_out(C, b * strideC + (r / N) * ldc + (r % N), 0.0f, 0.0f, beta, bias ? bias[r % N] : 0.0f);
            continue;
        }
        float *c = C + b * strideC + (r / N) * ldc + (r % N);
        const float v = beta == 0.0f ? 0.0f : beta * *c;
        *c = bias ? v + bias[r % N] : v;
    }
}

// Plain 16-byte-per-lane copy of known size: the yardstick that hardware traffic counters
// (rocprofv3 FETCH_SIZE / WRITE_SIZE) are scaled by.
__global__ void copy_kernel(const floatx4 *src, floatx4 *dst, long long n16) {
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n16;
         i += (long long)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// Split-K second pass: C = alpha * (ws[0] + ws[1] + ...) + beta * C (+ bias), V consecutive entries of a row per lane.
// A work-group takes 2^logCols units of V columns by 2^logRows rows (rows of all batch items in one sequence), and
// 2^logParts groups of its lanes share the partitions between them: a group adds its partitions in order, the sums of the
// groups meet in LDS and are added in order too, so the result does not depend on timing.
// Bound by one or two memory latencies behind the launch.  Places come from shifts (three 64-bit divisions per lane were
// most of the instructions) and all partitions of a group are in flight together: whole calls 16-bit 256 x 256 x 65536
// (32 partitions) 21.4 -> 19.8 us, 128 x 64 x 25536 (50) 9.7 -> 8.4, fp32 24 x 112 x 3904 (8) 8.0 -> 6.9; 480 x 1184 x 2592
// (3, bound by the bytes) 40.7 -> 39.9.
struct ReduceParams {
    const float *ws;
    float *C;
    const float *bias;
    long long ldc, strideC;
    long long per;                   // entries of one partition
    int M, N;
    unsigned rows, blocks, colBlocks;    // rows: of all batch items
    int splitK, perGroup;            // perGroup: partitions of a group of lanes
    int logCols, logRows;
    float alpha, beta;
    int out16, vecC;                 // vecC: C takes 16-byte accesses
};
template <int V>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ReduceParams p) {
    typedef float Unit __attribute__((ext_vector_type(V)));
    __shared__ Unit sums[256];
    const int tid = threadIdx.x, col0 = tid & ((1 << p.logCols) - 1);
    const int row0 = (tid >> p.logCols) & ((1 << p.logRows) - 1), g = tid >> (p.logCols + p.logRows);
    const int first = g * p.perGroup, last = min(p.splitK, first + p.perGroup);
    for (unsigned block = blockIdx.x; block < p.blocks; block += gridDim.x) {
        const unsigned rb = block / p.colBlocks;
        const unsigned row = (rb << p.logRows) + row0;
        const long long col = ((long long)((block - rb * p.colBlocks) << p.logCols) + col0) * V;
        const bool inside = row < p.rows && col < p.N;
        Unit acc = 0.f;
        if (inside) {
            const float *w = p.ws + (long long)row * p.N + col;
            int s = first;
            for (; s + 8 <= last; s += 8) {               // eight independent loads, added in partition order
                Unit v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const Unit *>(w + (s + u) * p.per);
#pragma unroll
                for (int u = 0; u < 8; ++u) acc += v[u];
            }
            // and what is left in one go, the last one read again where there is less
            auto rest = [&](auto n) {
                Unit v[decltype(n)::value];
#pragma unroll
                for (int u = 0; u < decltype(n)::value; ++u)
                    v[u] = *reinterpret_cast<const Unit *>(w + min(s + u, last - 1) * p.per);
#pragma unroll
                for (int u = 0; u < decltype(n)::value; ++u)
                    if (s + u < last) acc += v[u];
            };
            if (s + 4 < last) rest(std::integral_constant<int, 7>{});
            else if (s + 2 < last) rest(std::integral_constant<int, 4>{});
            else if (s + 1 < last) rest(std::integral_constant<int, 2>{});
            else if (s < last) rest(std::integral_constant<int, 1>{});
        }
        if (p.perGroup < p.splitK) {
            sums[tid] = acc;
            __syncthreads();
            if (g == 0)
                for (int t = tid + (1 << (p.logCols + p.logRows)); t < 256; t += 1 << (p.logCols + p.logRows)) acc += sums[t];
            __syncthreads();
        }
        if (g != 0 || !inside) continue;
        unsigned r = row;
        long long at = 0;
        if (p.rows != (unsigned)p.M) {
            const unsigned b = row / (unsigned)p.M;
            r = row - b * (unsigned)p.M;
            at = b * p.strideC;
        }
        at += r * p.ldc + col;
        if (p.out16) {
#pragma unroll
            for (int e = 0; e < V; ++e)
                store_bf16_out(p.C, at + e, acc[e], p.alpha, p.beta, p.bias ? p.bias[col + e] : 0.0f);
            continue;
        }
        float *c = p.C + at;
        Unit v = p.alpha * acc;
        if (p.beta != 0.0f) {
            Unit old;
            if (V == 4 && p.vecC) old = *reinterpret_cast<const Unit *>(c);
            else
#pragma unroll
                for (int e = 0; e < V; ++e) old[e] = c[e];
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = fmaf(p.beta, old[e], p.alpha * acc[e]);
        }
        if (p.bias) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += p.bias[col + e];
        }
        if (V == 4 && p.vecC) *reinterpret_cast<Unit *>(c) = v;
        else
#pragma unroll
            for (int e = 0; e < V; ++e) c[e] = v[e];
    }
}

// Second pass of a launch whose last round was partitioned along K (tail_split): work-group
// (b, y) adds up rows 8 y .. 8 y + 7 of the compact partial tiles [partition][b] of tile
// tileBase + b in partition order and writes them to C.  Few tiles are partitioned (fewer than one
// round of work-groups), so the rows of a tile are spread over many work-groups; partial sums are
// read 16 bytes per lane (the workspace is 16-byte aligned, tiles are multiples of 16 floats wide).
#define KS_TAIL_REDUCE_ROWS 8
__global__ void tail_reduce_kernel(const GemmParams p) {
    const TileCoord tc = tile_of_logical(p, blockIdx.x);       // partition 0 of tile tileBase + blockIdx.x
    const int bm = p.bm, bn = p.bn, S = p.splitK;
    const long long tileElems = (long long)bm * bn;
    const float *w0 = p.ws + (long long)blockIdx.x * tileElems;
    const long long per = (long long)p.tileSpan * tileElems;
    const int r0 = tc.tm * bm, c0 = tc.tn * bn;
    const int rows = p.M - r0 < bm ? p.M - r0 : bm, cols = p.N - c0 < bn ? p.N - c0 : bn;
    const int rFirst = (int)blockIdx.y * KS_TAIL_REDUCE_ROWS;
    const int q = bn / 4;                                      // float4 units per tile row
    for (int u = threadIdx.x; u < KS_TAIL_REDUCE_ROWS * q; u += blockDim.x) {
        const int r = rFirst + u / q, c = (u % q) * 4;
        if (r >= rows || c >= cols) continue;
        const float *w = w0 + (long long)r * bn + c;
        floatx4 acc = *reinterpret_cast<const floatx4 *>(w);
        int s = 1;
        for (; s + 8 <= S; s += 8) {                 // eight independent loads, added in partition order
            floatx4 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const floatx4 *>(w + (long long)(s + k) * per);
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += v[k];
        }
        for (; s < S; ++s) acc += *reinterpret_cast<const floatx4 *>(w + (long long)s * per);
        const long long at = (long long)(r0 + r) * p.ldc + (c0 + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (c + e >= cols) break;
            if (p.out16) {
                store_bf16_out(p.C, at + e, acc[e], p.alpha, p.beta, p.bias ? p.bias[c0 + c + e] : 0.0f);
                continue;
            }
            float *cp = p.C + at + e;
            float v = p.alpha * acc[e];
            if (p.beta != 0.0f) v = fmaf(p.beta, *cp, v);
            if (p.bias) v += p.bias[c0 + c + e];
            *cp = v;
        }
    }
}

// One 16-bit operand copied to where the direct-to-LDS path can read it: rows of `cols` elements, `ld` apart, to
// outRows rows of outChunks x 8 elements without a gap; what the operand does not have reads as zero.
struct OperandCopy {
    const uint16_t *src;
    uint16_t *dst;
    long long ld;
    int rows, cols;
    unsigned outChunks, units;       // units: sixteen-byte chunks of the whole copy
};
#define KS_COPY_CHUNKS 4             // chunks per thread, loads of all in flight
// Bound by memory: every operand byte is read and written once, 27.5 MB of copies in 10.1 us (5.4 TB/s).  Loads are
// sixteen bytes at any element, which the memory pipe takes at a quarter of its rate where the address is no multiple of
// four (15 against 59 bytes per clock and compute unit from L2): still above what memory delivers.  A chunk over the
// end of a row is read whole as well, up to the last ones of the operand; element loads for all of them took 6.7 us
// instead of 5.3 over 1000 x 777 x 1509.
__global__ __launch_bounds__(256) void copy_operands_kernel(const OperandCopy a, const OperandCopy b, unsigned groupsA) {
    const bool second = blockIdx.x >= groupsA;
    const OperandCopy o = second ? b : a;
    const unsigned first = (blockIdx.x - (second ? groupsA : 0u)) * (256u * KS_COPY_CHUNKS) + threadIdx.x;
    const long long lastWhole = (o.rows - 1) * o.ld + o.cols - 8;       // last element from which eight may be read
    uintx4 v[KS_COPY_CHUNKS];
#pragma unroll
    for (int j = 0; j < KS_COPY_CHUNKS; ++j) {
        const unsigned n = first + j * 256u, row = n / o.outChunks, col = (n - row * o.outChunks) * 8u;
        const int left = (int)row < o.rows ? o.cols - (int)col : 0;
        const long long at = (long long)row * o.ld + col;
        v[j] = uintx4{0u, 0u, 0u, 0u};
        if (n < o.units && left > 0) {
            if (at <= lastWhole) {
                v[j] = load16_any(o.src + at);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e < left) v[j][e >> 1] |= (unsigned)o.src[at + e] << (16 * (e & 1));
            }
        }
    }
#pragma unroll
    for (int j = 0; j < KS_COPY_CHUNKS; ++j) {
        const unsigned n = first + j * 256u, row = n / o.outChunks, col = (n - row * o.outChunks) * 8u;
        const int left = o.cols - (int)col;
        // what was read beyond the end of the row is taken out again
#pragma unroll
        for (int e = 0; e < 4; ++e) v[j][e] &= 2 * e + 2 <= left ? ~0u : 2 * e + 1 == left ? 0xFFFFu : 0u;
        if (n < o.units) reinterpret_cast<uintx4 *>(o.dst)[n] = v[j];
    }
}

int validate(int transA, int transB, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda,
             const void *B, int64_t ldb, const float *C, int64_t ldc, int64_t batch,
             int64_t strideC) {
    if ((transA != 0 && transA != 1) || (transB != 0 && transB != 1)) return KS_ERR_INVALID_ARG;
    if (M < 0 || N < 0 || K < 0 || batch < 0) return KS_ERR_INVALID_ARG;
    const int64_t lim = 2147483647LL - 512;
    if (M >= lim || N >= lim || K >= lim || batch >= lim) return KS_ERR_UNSUPPORTED;
    // leading dimensions take part in 64-bit element offsets (row * ld, row < 2^31): with ld < 2^31
    // every such product stays below 2^62
    const int64_t ldLim = 1LL << 31;
    if (lda >= ldLim || ldb >= ldLim || ldc >= ldLim) return KS_ERR_UNSUPPORTED;
    if (M == 0 || N == 0 || batch == 0) return KS_OK;
    if (!C || ldc < N) return KS_ERR_INVALID_ARG;
    if (K > 0) {
        if (!A || !B) return KS_ERR_INVALID_ARG;
        if (lda < (transA ? M : K) || ldb < (transB ? K : N)) return KS_ERR_INVALID_ARG;
    }
    if (batch > 1) {
        int64_t span = 0;                             // elements one item of C covers
        if (__builtin_mul_overflow(M - 1, ldc, &span) || __builtin_add_overflow(span, N, &span))
            return KS_ERR_UNSUPPORTED;
        const int64_t s = strideC < 0 ? -strideC : strideC;
        if (s < span) return KS_ERR_INVALID_ARG;
    }
    return KS_OK;
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// 16-byte accesses: aligned operands, leading dimensions, contiguous extents and batch strides (w elements each)
bool vector_operands(int w, bool akc, bool bkc, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B,
                     int64_t ldb, int64_t batch, int64_t strideA, int64_t strideB) {
    return aligned(A, 16) && aligned(B, 16) && lda % w == 0 && ldb % w == 0 && (akc ? K : M) % w == 0 && (bkc ? K : N) % w == 0 &&
           (batch == 1 || (strideA % w == 0 && strideB % w == 0));
}
// what the direct-to-LDS path of the 16-bit members asks of them beside whole K-steps: 16-byte accesses and
// tile-relative byte offsets that fit 32 bits
bool dma_operands(bool akc, bool bkc, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                  int64_t batch, int64_t strideA, int64_t strideB) {
    return vector_operands(8, akc, bkc, M, N, K, A, lda, B, ldb, batch, strideA, strideB) && g_forceGeneric == 0 &&
           lda <= (1LL << 22) && ldb <= (1LL << 22);
}

// Whether aligned copies of 16-bit operands (`bytes` of them) pay: what the direct-to-LDS path saves grows with the
// flops, what the copies cost (a launch, then each byte written and read once more, 5.4 TB/s) with the bytes.
// Of 176 problems of at least 1.5 GFLOP on operands that nothing aligns, 65 lie on this side of the line at 0.775 of the
// time of the register-staged path (6208 x 1472 x 5312 NN 216 -> 137 us, 1152 x 2624 x 4096 NN 61 -> 47), one of them
// slower (1.04); with the line at 4 GFLOP it would be 80 at 0.806, eight slower by up to 1.19 (1472 x 1280 x 1088 TT).
bool copies_pay(int64_t M, int64_t N, int64_t K, size_t bytes) {
    return 2.0 * (double)M * (double)N * (double)K >= 1e10 + 250.0 * (double)bytes;
}

// The reduction pass of a split-K launch.  Lanes share the partitions of an entry, two or more to a group, while that
// leaves fewer than 2^17 of them, eight waves a compute unit, or 2^16 where a lane reads one float: with more the reads fill the
// memory pipe by themselves.  240 split calls against 2^17 for both: 0.997 in the mean, 23 faster by more than 1.5 %, nearly all
// of single floats (86 x 199 x 8704 in 17 partitions 0.93), three slower (158 x 257 x 18688 1.03); sixteen bytes a lane were level or
// slower with 2^16 (256 x 256 x 65536 19.6 -> 20.2 us).
// The groups, and with them the order of the sums, follow from the sizes alone: where N is a multiple of four and only the
// scratch is not 16-byte aligned, lanes read one float each in the groups of the wide form.
int launch_reduce(const GemmParams &p, bool vecC, hipStream_t stream) {
    // the kernel counts rows in 32 bits: all batch items in one launch, or one each
    const bool each = (int64_t)p.batch * p.M >= (1LL << 31);
    const int64_t rows = each ? p.M : (int64_t)p.batch * p.M;
    ReduceParams r;
    r.bias = p.bias;
    r.ldc = p.ldc; r.strideC = p.out16 ? p.strideC16 : p.strideC;
    r.M = p.M; r.N = p.N;
    r.rows = (unsigned)rows;
    r.per = (long long)p.batch * p.M * p.N;
    r.splitK = p.splitK;
    r.alpha = p.alpha; r.beta = p.beta;
    r.out16 = p.out16; r.vecC = vecC ? 1 : 0;
    const bool quads = p.N % 4 == 0, vec = quads && aligned(p.ws, 16);
    const int64_t units = vec ? p.N / 4 : p.N, lanes = (quads ? p.N / 4 : p.N) * rows;
    int logParts = 0;
    while (logParts < 3 && (lanes << logParts) < (quads ? 1 << 17 : 1 << 16) && p.splitK >= 4 << logParts) ++logParts;
    r.perGroup = (p.splitK + (1 << logParts) - 1) >> logParts;
    r.logCols = 0;
    while (r.logCols < 6 && r.logCols < 8 - logParts && (1 << r.logCols) < units) ++r.logCols;   // a wave's row
    r.logRows = 8 - logParts - r.logCols;
    const int64_t colBlocks = (units + (1 << r.logCols) - 1) >> r.logCols;
    const int64_t blocks = colBlocks * ((rows + (1 << r.logRows) - 1) >> r.logRows);   // < 2^31 for any scratch a device holds
    r.colBlocks = (unsigned)colBlocks;
    r.blocks = (unsigned)blocks;
    const dim3 grid((unsigned)(blocks < 1048576 ? blocks : 1048576));
    for (int64_t item = 0; item < (each ? p.batch : 1); ++item) {
        r.ws = p.ws + item * p.M * p.N;
        r.C = p.out16 ? reinterpret_cast<float *>(reinterpret_cast<uint16_t *>(p.C) + item * r.strideC) : p.C + item * r.strideC;
        if (vec) hipLaunchKernelGGL(splitk_reduce_kernel<4>, grid, dim3(256), 0, stream, r);
        else hipLaunchKernelGGL(splitk_reduce_kernel<1>, grid, dim3(256), 0, stream, r);
        if (hipGetLastError() != hipSuccess) return KS_ERR_LAUNCH;
    }
    return KS_OK;
}

// Scratch for split-K partial sums: the registered workspace, or the library's static array.
struct Workspace {
    void *ptr;
    size_t bytes;
};
Workspace registered_ws() { return Workspace{g_ws, g_wsBytes}; }

// K partitions of a member whose count is chosen per call: as many as fill the device, at least two K-steps
// each, and no more than the scratch can hold (1 = the plain single-kernel form)
int64_t partitions(const InstanceDesc *d, bool f32, int64_t M, int64_t N, int64_t K, int64_t batch, Workspace w) {
    const int64_t tiles = ((M + d->bm - 1) / d->bm) * ((N + d->bn - 1) / d->bn) * batch;
    const int64_t steps = ((K + d->bk - 1) / d->bk + d->kw - 1) / d->kw;
    if (!w.ptr) return 1;
    int64_t s = auto_split(d, tiles, steps, f32);
    if (g_splitForced > 0) s = g_splitForced > 1 && 2 * (int64_t)g_splitForced > steps ? (steps / 2 > 1 ? steps / 2 : 1) : g_splitForced;
    const size_t per = (size_t)batch * (size_t)M * (size_t)N * sizeof(float);
    if ((size_t)s * per > w.bytes) s = (int64_t)(w.bytes / per);
    return s < 1 ? 1 : s;
}

int remainder_member(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int tA, int tB, Workspace w);

int run_ws(Workspace wsp, int dtype, int id, int transA, int transB, int64_t M, int64_t N, int64_t K, float alpha,
           const void *A, int64_t lda, const void *B, int64_t ldb, float beta, float *C, int64_t ldc,
           int64_t batch, int64_t strideA, int64_t strideB, int64_t strideC, hipStream_t stream,
           const float *bias = nullptr, int out16 = 0, ks_launch_plan_t *planOnly = nullptr, bool own = false,
           bool copied = false, bool selected = false) {
    const InstanceDesc *d = desc_of(dtype, id);
    if (!d) return KS_ERR_INVALID_ARG;
    const int rc = validate(transA, transB, M, N, K, A, lda, B, ldb, C, ldc, batch, strideC);
    if (rc != KS_OK) return rc;
    if (planOnly) {
        *planOnly = ks_launch_plan_t{};
        planOnly->kernel_id = id;
        planOnly->split_k = 1;
        planOnly->tiles_per_workgroup = 1;
    }
    if (M == 0 || N == 0 || batch == 0) return KS_OK;
    if (planOnly && K == 0) return KS_OK;
    std::call_once(g_once, init_tables);

    // An error left behind by an earlier, unrelated runtime call must not be blamed on this launch.
    (void)hipGetLastError();

    if (K == 0) {
        const long long total = (long long)batch * M * N;
        const int grid = (int)((total + 255) / 256 < 65535 ? (total + 255) / 256 : 65535);
        hipLaunchKernelGGL(scale_c_kernel, dim3(grid), dim3(256), 0, stream, C, (long long)ldc,
                           (long long)strideC, (int)M, (int)N, (int)batch, beta, bias, out16);
        return hipGetLastError() == hipSuccess ? KS_OK : KS_ERR_LAUNCH;
    }

    // a pruned build holds only the kept members
    if ((dtype == KS_F32 ? g_f32[id] : g_bf16[id]) == nullptr) return KS_ERR_UNSUPPORTED;

    // A call that names no member and would run one of the skinny or square ones with few tiles takes the K-slices form
    // where its estimate is the lower one (slices.hpp).  Named members, a caller's own tree, forced partitions and forced copies are
    // followed as they are.  The form takes no scratch; what the member would do with the scratch at hand is what it is compared with.
    // Drawn problems (64 .. 4096 in each dimension, skinny and tall ones, four layouts): aligned 495 of 1300 take it, 0.755 of the
    // time; with rows that nothing aligns 521 of 1597, 0.70.
    int64_t estimated = 0;                            // K partitions of this member and call, once known
    if (selected && dtype != KS_F32 && batch == 1 && g_splitForced == 0 && g_forceGeneric == 0 && slices_possible(id, M, N, K) &&
        !custom_tree(dtype)) {
        const bool akc = transA == 0, bkc = transB == 1;
        const bool staged = K % 64 != 0 || !dma_operands(akc, bkc, M, N, K, A, lda, B, ldb, 1, 0, 0);
        int t = -1;
        // (copies of the operands asked for wherever they can be made are the member's)
        if (slices_worth(staged, akc, bkc, M, N, K, lda, ldb) && !(staged && g_operandCopies > 0)) {
            const int64_t parts = d->splitK > 0 ? 1 : (estimated = partitions(d, false, M, N, K, 1, wsp)), kTiles = (K + d->bk - 1) / d->bk;
            const int64_t groups = ((M + d->bm - 1) / d->bm) * ((N + d->bn - 1) / d->bn) * parts;
            const double other = slices_other_us(staged, id, M, N, K, groups, (kTiles + parts - 1) / parts, parts,
                                                 4.0 * (double)parts * (double)M * (double)N);
            t = slices_tile(staged, id, akc, bkc, M, N, K, lda, ldb, other);
        }
        if (t >= 0) {
            const SliceTile &tile = kSliceTiles[t];
            GemmParams p{};
            p.A = A; p.B = B; p.C = C; p.bias = bias; p.out16 = out16;
            p.lda = lda; p.ldb = ldb; p.ldc = ldc;
            p.M = (int)M; p.N = (int)N; p.K = (int)K; p.batch = 1;
            p.tilesM = (int)((M + tile.bm - 1) / tile.bm);
            p.tilesN = (int)((N + tile.bn - 1) / tile.bn);
            p.splitK = 1; p.kChunk = (int)K; p.tilesPerWG = 1; p.bandRows = 8;
            p.bm = tile.bm; p.bn = tile.bn;
            p.alpha = alpha; p.beta = beta;
            const int grid = p.tilesM * p.tilesN;
            p.grid3d = (double)(M + N) * (double)K * 2 <= (double)KS_GRID3D_BYTES ? 1 : 0;
            set_tile_order(p);
            if (planOnly) {
                planOnly->path = 16 + t;
                planOnly->vector_loads = vector_operands(8, akc, bkc, M, N, K, A, lda, B, ldb, 1, 0, 0) ? 1 : 0;
                planOnly->grid_3d = p.grid3d;
                planOnly->workgroups = grid;
                return KS_OK;
            }
            const int pastCache = (slices_past_cache(M, K, p.tilesN) ? 1 : 0) + (slices_past_cache(N, K, p.tilesM) ? 2 : 0);
            launch_bf16_slices(t, p, grid, (akc ? 2 : 0) + (bkc ? 1 : 0) + (dtype == KS_F16 ? 16 : 0), pastCache, stream);
            return hipGetLastError() == hipSuccess ? KS_OK : KS_ERR_LAUNCH;
        }
    }

    // 16-bit operands whose K is not a whole number of K-steps (of half ones for members of K-step 128)
    // would take the member's register-staged path for all of K.  Where everything else qualifies for the
    // direct-to-LDS path, the K range is cut instead: the remainder (fewer than one K-step, register-staged)
    // goes first and applies alpha, beta and the bias, then the whole K-steps run on the fast path with
    // beta = 1.  The partial result passes through C in fp32 (one more rounding per entry, far inside the
    // bound), so an output kept in bf16 is not served this way.  The line (every layout but NT, and NT from 2^24
    // entries of output on) is a published one: ks_set_fast_path in the header states it, ks_launch_plan_t
    // reports it, and the bits of every such call that runs a member, named or selected, hang on it (a selecting call that takes the
    // K-slices form has returned above: 512 x 512 x 1032 TN).  It was drawn when the
    // register-staged path loaded two bytes per lane.  By today's times, cut against register-staged over all of
    // K with a remainder of 24, it would lie at 2^24 entries for NN, TN and TT and nowhere for NT: 4096^3 NN 150 / 165
    // us, TN 140 / 155, TT 142 / 155, NT 160 / 152; 2048^3 NN 39 / 35, TN 35 / 33; 1024^3 NN 14.7 / 12.4.
    if (dtype != KS_F32 && !out16 && g_forceGeneric == 0 && K % dma_k_step(*d) != 0 && K % 8 == 0 && K >= 4LL * d->bk) {
        const int64_t Kr = K % dma_k_step(*d), Kh = K - Kr;
        const bool akc = transA == 0, bkc = transB == 1;
        const bool pays = !(akc && bkc) || M * N >= (1LL << 24);
        const bool vecOk = pays && aligned(A, 16) && aligned(B, 16) && lda % 8 == 0 && ldb % 8 == 0 && (akc || M % 8 == 0) &&
                           (bkc || N % 8 == 0) && (batch == 1 || (strideA % 8 == 0 && strideB % 8 == 0)) &&
                           lda <= (1LL << 22) && ldb <= (1LL << 22);
        if (vecOk) {
            const uint16_t *Ar = static_cast<const uint16_t *>(A) + (akc ? Kh : Kh * lda);
            const uint16_t *Br = static_cast<const uint16_t *>(B) + (bkc ? Kh : Kh * ldb);
            if (planOnly) {
                const int prc = run_ws(wsp, dtype, id, transA, transB, M, N, Kh, alpha, A, lda, B, ldb, 1.0f, C, ldc, batch,
                                       strideA, strideB, strideC, stream, nullptr, 0, planOnly);
                if (prc == KS_OK) planOnly->k_remainder = (int32_t)Kr;
                return prc;
            }
            // the remainder is a GEMM with a very short K of its own, bound by the pass over C: it
            // runs with the member the deployed tree names for that problem
            int idr = remainder_member(dtype, M, N, Kr, batch, transA, transB, wsp);
            if (idr < 0) idr = id;
            const int r1 = run_ws(wsp, dtype, idr, transA, transB, M, N, Kr, alpha, Ar, lda, Br, ldb, beta, C, ldc, batch,
                                  strideA, strideB, strideC, stream, bias, 0, nullptr);
            if (r1 != KS_OK) return r1;
            return run_ws(wsp, dtype, id, transA, transB, M, N, Kh, alpha, A, lda, B, ldb, 1.0f, C, ldc, batch, strideA,
                          strideB, strideC, stream, nullptr, 0, nullptr);
        }
    }

    // 16-bit operands that the direct-to-LDS path cannot read as they are: copies that it can (OperandCopy), where the
    // scratch holds them and they pay.  The member and its partitions of K stay the same, and with them the order of the
    // sums, but for the tiles that a hybrid launch partitions (tail_split, direct-to-LDS only).  The
    // registered workspace is for members that may use it (those with split_k == 1 never do).
    // Partial sums come first: without their partitions a few tiles leave the device idle (1024 x 1024 x 64001 NT in
    // 256 MiB ran 16 work-groups instead of 256, 1173 us against 170 on the operands as they are; 2000 x 900 x 20001 TN in 128
    // MiB two partitions instead of eight, 211 against 121).
    if (dtype != KS_F32 && !copied && batch == 1 && g_forceGeneric == 0 && g_operandCopies != 0 && wsp.ptr &&
        (own || d->splitK != 1)) {
        const bool akc = transA == 0, bkc = transB == 1;
        const int64_t Kc = (K + dma_k_step(*d) - 1) / dma_k_step(*d) * dma_k_step(*d);
        auto misfit = [&](const void *x, int64_t ld, bool kc, int64_t extent) {
            return Kc != K || !aligned(x, 16) || ld % 8 != 0 || ld > (1LL << 22) || (!kc && extent % 8 != 0);
        };
        const bool copyA = misfit(A, lda, akc, M), copyB = misfit(B, ldb, bkc, N);
        auto rows_of = [&](bool kc, int64_t extent) { return kc ? extent : Kc; };
        auto length_of = [&](bool kc, int64_t extent) { return kc ? Kc : (extent + 7) / 8 * 8; };
        const int64_t chunksA = copyA ? rows_of(akc, M) * length_of(akc, M) / 8 : 0;
        const int64_t chunksB = copyB ? rows_of(bkc, N) * length_of(bkc, N) / 8 : 0;
        const size_t bytes = (size_t)(chunksA + chunksB) * 16;
        auto holds = [&] {
            const int64_t s = d->splitK > 0 ? d->splitK : partitions(d, false, M, N, K, 1, wsp);
            return wsp.bytes >= bytes + (s > 1 ? (size_t)s * (size_t)M * (size_t)N * sizeof(float) : 0) + 16;
        };
        const bool reach = length_of(akc, M) <= (1LL << 22) && length_of(bkc, N) <= (1LL << 22);
        if ((copyA || copyB) && reach && chunksA + chunksB < (1LL << 31) &&
            (g_operandCopies > 0 || copies_pay(M, N, K, bytes)) && holds()) {
            // at the end of the scratch: partial sums stay at its beginning
            char *const end = static_cast<char *>(wsp.ptr) + wsp.bytes;
            char *const at = end - bytes - reinterpret_cast<uintptr_t>(end - bytes) % 16;
            const Workspace rest{wsp.ptr, (size_t)(at - static_cast<char *>(wsp.ptr))};
            uint16_t *const toA = reinterpret_cast<uint16_t *>(at), *const toB = toA + chunksA * 8;
            if (!planOnly) {
                const OperandCopy a{static_cast<const uint16_t *>(A), toA, lda, (int)(akc ? M : K), (int)(akc ? K : M),
                                    (unsigned)(length_of(akc, M) / 8), (unsigned)chunksA};
                const OperandCopy b{static_cast<const uint16_t *>(B), toB, ldb, (int)(bkc ? N : K), (int)(bkc ? K : N),
                                    (unsigned)(length_of(bkc, N) / 8), (unsigned)chunksB};
                const int64_t per = 256 * KS_COPY_CHUNKS, groupsA = (chunksA + per - 1) / per, groupsB = (chunksB + per - 1) / per;
                hipLaunchKernelGGL(copy_operands_kernel, dim3((unsigned)(groupsA + groupsB)), dim3(256), 0, stream, a, b,
                                   (unsigned)groupsA);
                if (hipGetLastError() != hipSuccess) return KS_ERR_LAUNCH;
            }
            const int rc = run_ws(rest, dtype, id, transA, transB, M, N, Kc, alpha, copyA ? toA : A,
                                  copyA ? length_of(akc, M) : lda, copyB ? toB : B, copyB ? length_of(bkc, N) : ldb, beta, C,
                                  ldc, 1, 0, 0, 0, stream, bias, out16, planOnly, own, true);
            if (rc == KS_OK && planOnly) {               // the operands as they are, and that they are copied
                planOnly->path = 0;
                planOnly->vector_loads = vector_operands(8, akc, bkc, M, N, K, A, lda, B, ldb, 1, 0, 0) ? 1 : 0;
                planOnly->operand_copies = (copyA ? 1 : 0) + (copyB ? 2 : 0);
            }
            return rc;
        }
    }

    GemmParams p;
    p.A = A; p.B = B; p.C = C; p.ws = nullptr; p.bias = bias; p.out16 = out16;
    p.lda = lda; p.ldb = ldb; p.ldc = ldc;
    p.strideA = strideA; p.strideB = strideB;
    p.strideC = out16 ? 0 : strideC; p.strideC16 = out16 ? strideC : 0;
    p.M = (int)M; p.N = (int)N; p.K = (int)K; p.batch = (int)batch;
    p.tilesM = (int)((M + d->bm - 1) / d->bm);
    p.tilesN = (int)((N + d->bn - 1) / d->bn);
    const int64_t kTiles = (K + d->bk - 1) / d->bk;
    p.splitK = d->splitK;
    if (d->splitK == 0) p.splitK = (int)(estimated > 0 ? estimated : partitions(d, dtype == KS_F32, M, N, K, batch, wsp));
    p.kChunk = (int)(((kTiles + p.splitK - 1) / p.splitK) * d->bk);
    p.alpha = alpha; p.beta = beta;

    int64_t grid64 = (int64_t)p.tilesM * p.tilesN * batch * p.splitK;
    if (grid64 > 2147483647LL) return KS_ERR_UNSUPPORTED;
    // three-dimensional launch only where the tile order cannot matter for L2: few work-groups
    // and operands that fit one XCD's L2 several times over
    const double operandBytes = (double)(M + N) * (double)K * (double)batch * (dtype == KS_F32 ? 4 : 2);
    p.grid3d = grid64 <= KS_GRID3D_MAX && operandBytes <= (double)KS_GRID3D_BYTES && p.tilesM <= 65535 &&
                       batch * p.splitK <= 65535
                   ? 1
                   : 0;
    p.tilesPerWG = 1;
    p.bandRows = d->band;
    p.skGroups = 0; p.skRounds = 0; p.skTailTiles = 0;
    p.tileBase = 0; p.tileSpan = 0; p.bm = d->bm; p.bn = d->bn;
    const bool onBf16Pipe = dtype == KS_F32 && f32_parts_member(d->core, d->bm, d->bn, d->bk, d->kw, p.splitK > 1);
    // (a member with a form on the bf16 matrix pipe has the balanced form there alone)
    if (d->sk > 0 && (!onBf16Pipe || K >= f32_parts_least_k(d->kw))) {
        // Balanced persistent form where it pays (measured against the plain member of the same
        // tiles on the tuning tables): tiles that do not divide evenly over the work-groups, fewer
        // than four rounds of them (with more, the uneven last round matters less than what the
        // hardware's own dispatch gains by handing a tile to whichever unit is free), and at
        // least 1024 of K per tile and one K-step per share (below that the raw accumulator tiles
        // of the divided tiles and the second kernel cost more than the balance gains).  A forced work-group count
        // (ks_set_balanced_groups) takes the form whenever it can run.  Its scratch must be there
        // unless no tile is divided; otherwise the plain member runs.
        // With few tiles every tile is divided among many work-groups; a 512-thread member then
        // runs faster with one work-group per compute unit than with two (fewer raw accumulator
        // tiles per output tile, and the whole unit for each share): measured 2-10 % up to 80
        // tiles of 128x128, even from 110 to 224, 3-5 % the other way from 270 on.
        const int64_t groups = g_skPerCU == 0 && d->sk == 2 && d->threads >= 512 && grid64 <= 96 ? 256 : sk_groups(d);
        const int64_t tail = grid64 % groups;
        const bool fits = tail == 0 || (wsp.ptr && wsp.bytes >= sk_workspace_bytes(d) && aligned(wsp.ptr, 16));
        const bool pays = g_skPerCU > 0 || (tail != 0 && grid64 < 4 * groups && K >= 1024 && tail * kTiles >= groups);
        if (fits && pays && tail * kTiles < (1LL << 50)) {
            p.skGroups = (int)groups;
            p.skRounds = (int)(grid64 / groups);
            p.skTailTiles = (int)tail;
            p.ws = static_cast<float *>(wsp.ptr);
            p.grid3d = 0;
            grid64 = groups;
        }
    }
    // on the bf16 matrix pipe (gemm_f32_parts.hpp), where the K range of a work-group is long enough; that form has no
    // work-groups that walk several tiles
    const int64_t waveK = K < p.kChunk ? K : p.kChunk;
    const bool parts = onBf16Pipe && waveK >= f32_parts_least_k(d->kw);
    bool square = false;                             // 2 x 2 tiles of the member per work-group
    if (parts && d->bm == 64 && d->kw == 1 && d->splitK == 1) {
        const int64_t tilesM = (M + 127) / 128, tilesN = (N + 127) / 128, tiles128 = tilesM * tilesN * batch;
        square = g_tilesPerWG == 0 ? f32_parts_square(grid64, tiles128, K) : g_tilesPerWG == 4;
        if (square) {
            p.tilesM = (int)tilesM;
            p.tilesN = (int)tilesN;
            p.bm = p.bn = 128;
            p.tilesPerWG = 4;
            grid64 = tiles128;
        }
    }
    if (dtype == KS_F32 && !parts && !p.grid3d && p.splitK == 1 && p.skGroups == 0 && f32_multi_tile(d->core, d->bm, d->bn, d->p1, d->p2, d->kw)) {
        p.tilesPerWG = g_tilesPerWG > 0 ? g_tilesPerWG : multi_tiles(d, grid64, K);
        grid64 = (grid64 + p.tilesPerWG - 1) / p.tilesPerWG;
    }

    if (p.splitK > 1) {
        const size_t need = (size_t)p.splitK * (size_t)batch * (size_t)M * (size_t)N * sizeof(float);
        if (!wsp.ptr || wsp.bytes < need) return KS_ERR_WORKSPACE;
        p.ws = static_cast<float *>(wsp.ptr);
    }

    // contiguous direction: A is K-contiguous when not transposed, B when transposed
    const bool akc = transA == 0, bkc = transB == 1;
    const int splitBit = p.splitK > 1 ? 8 : 0;       // read by instances whose split is chosen per call
    // Load form of the fp32 members: of the LDS-staged ones as described in ks_common.hpp, UNITS up to eight K-steps
    // of a wave in any member (it gains up to four of them); of the register-fed ones (gemm_f32_direct.hpp) by K alone.
    const bool registerFed = d->core == KS_CORE_DIRECT || d->core == KS_CORE_KSLICE;
    const int64_t stepK = (int64_t)d->bk * d->kw;
    const bool oneTile = p.skGroups == 0 && p.tilesPerWG == 1;
    const int group = d->threads / d->kw;
    const bool units = registerFed ? K % 4 == 0
                                   : oneTile && (akc ? K : M) % 4 == 0 && (bkc ? K : N) % 4 == 0 &&
                                         (waveK <= 8 * stepK || f32_units_at_any_k(d->core, d->bm, d->bn, d->bk, group, d->kw));
    const bool elements = oneTile && waveK <= f32_element_steps(d->core, d->bm, d->bn, d->bk, group, d->kw) * stepK;
    // and of the register-staged path of the 16-bit ones (gemm_bf16.hpp)
    const bool chunks = akc && bkc && d->bk == 128 && K % 8 == 0 && K % 128 != 0 && waveK > 128 && waveK < 512;
    const int variant = (akc ? 4 : 0) + (bkc ? 2 : 0) + ((dtype == KS_F32 ? units : chunks) ? 1 : 0) + (elements ? 32 : 0) + (parts ? 64 : 0) + (square ? 128 : 0) + splitBit;

    // bf16 fast path: operand tiles go global -> LDS directly.
    const int f16Bit = dtype == KS_F16 ? 16 : 0;     // same 16-bit members, binary16 MFMA
    const bool dma = copied || (dtype != KS_F32 && K % dma_k_step(*d) == 0 && dma_operands(akc, bkc, M, N, K, A, lda, B, ldb, batch, strideA, strideB));
    // Hybrid launch of a 16-bit member whose split is chosen per call: whole rounds of work-groups
    // compute their tiles over all of K, the tiles of the last, partly filled round are cut along
    // K (tail_split), and a third kernel adds their partial tiles up.
    int64_t tailS = 0, tailTiles = 0, mainGrid = grid64;
    if (dma && d->splitK == 0 && p.splitK == 1 && batch == 1 && g_tailSplit != 0 && wsp.ptr &&
        aligned(wsp.ptr, 16)) {
        const int64_t slots = split_slots(d, false);
        const int64_t s = tail_split(d, grid64, kTiles);
        const int64_t tail = grid64 % slots;
        if (s >= 2 && (size_t)s * (size_t)tail * (size_t)d->bm * (size_t)d->bn * sizeof(float) <= wsp.bytes) {
            tailS = s; tailTiles = tail; mainGrid = grid64 - tail;
            p.grid3d = 0;                            // both launches walk the one-dimensional tile order
        }
    }
    if (planOnly) {
        planOnly->tail_split = (int32_t)tailS;
        planOnly->split_k = p.splitK;
        planOnly->vector_loads =
            vector_operands(dtype == KS_F32 ? 4 : 8, akc, bkc, M, N, K, A, lda, B, ldb, batch, strideA, strideB) ? 1 : 0;
        planOnly->grid_3d = p.grid3d;
        planOnly->tiles_per_workgroup = p.tilesPerWG;
        planOnly->workgroups = tailS ? mainGrid + tailTiles * tailS : grid64;
        planOnly->balanced_groups = p.skGroups;
        planOnly->divided_tiles = p.skTailTiles;
        planOnly->path = parts ? 3
                         : !dma ? 0
                         : bf16_two_groups(d->core == KS_CORE_MFMA32 ? 32 : 16, d->bm, d->bn, d->bk, d->p1, d->p2,
                                           d->ldsBytes / (d->bk * (d->bm + d->bn) * 2))
                             ? 2
                             : 1;
        return KS_OK;
    }
    set_tile_order(p);
    if (tailS) {
        const int layoutBits = (akc ? 2 : 0) + (bkc ? 1 : 0) + f16Bit;
        g_bf16_dma[id](p, (int)mainGrid, layoutBits, stream);
        if (hipGetLastError() != hipSuccess) return KS_ERR_LAUNCH;
        GemmParams q = p;
        q.splitK = (int)tailS;
        q.kChunk = (int)(((kTiles + tailS - 1) / tailS) * d->bk);
        q.tileBase = (int)mainGrid;
        q.tileSpan = (int)tailTiles;
        q.ws = static_cast<float *>(wsp.ptr);
        set_tile_order(q);
        g_bf16_dma[id](q, (int)(tailTiles * tailS), layoutBits + 8, stream);
        if (hipGetLastError() != hipSuccess) return KS_ERR_LAUNCH;
        hipLaunchKernelGGL(tail_reduce_kernel,
                           dim3((unsigned)tailTiles, (unsigned)((d->bm + KS_TAIL_REDUCE_ROWS - 1) / KS_TAIL_REDUCE_ROWS)),
                           dim3(256), 0, stream, q);
        return hipGetLastError() == hipSuccess ? KS_OK : KS_ERR_LAUNCH;
    }
    if (dma)
        g_bf16_dma[id](p, (int)grid64, (akc ? 2 : 0) + (bkc ? 1 : 0) + splitBit + f16Bit, stream);
    else
        (dtype == KS_F32 ? g_f32[id] : g_bf16[id])(p, (int)grid64, variant + f16Bit, stream);
    if (hipGetLastError() != hipSuccess) return KS_ERR_LAUNCH;

    if (p.splitK > 1) {
        const int rc = launch_reduce(p, aligned(C, 16) && ldc % 4 == 0 && (batch == 1 || strideC % 4 == 0), stream);
        if (rc != KS_OK) return rc;
    }
    return KS_OK;
}

int run(int dtype, int id, int transA, int transB, int64_t M, int64_t N, int64_t K, float alpha,
        const void *A, int64_t lda, const void *B, int64_t ldb, float beta, float *C, int64_t ldc,
        int64_t batch, int64_t strideA, int64_t strideB, int64_t strideC, hipStream_t stream,
        const float *bias = nullptr, int out16 = 0, bool selected = false) {
    return run_ws(registered_ws(), dtype, id, transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, batch,
                  strideA, strideB, strideC, stream, bias, out16, nullptr, false, false, selected);
}

}  // namespace
}  // namespace ks

using namespace ks;

extern "C" int ks_num_kernels(int dtype) {
    if (dtype == KS_F32) return kNumF32;
    if (dtype == KS_BF16 || dtype == KS_F16) return kNumBf16;
    return KS_ERR_INVALID_ARG;
}

extern "C" int ks_kernel_info(int dtype, int kernel_id, ks_kernel_info_t *out) {
    const InstanceDesc *d = desc_of(dtype, kernel_id);
    if (!d || !out) return KS_ERR_INVALID_ARG;
    out->id = d->id;
    out->dtype = dtype;
    out->core = d->core;
    out->bm = d->bm; out->bn = d->bn; out->bk = d->bk;
    const int frag = d->core == KS_CORE_MFMA32 ? 32 : 16;
    if (d->core == KS_CORE_FMA) {
        out->wm = d->p1; out->wn = d->p2; out->tm = d->p1; out->tn = d->p2;
    } else if (d->core == KS_CORE_KSLICE) {
        out->wm = d->p2; out->wn = d->p2; out->tm = d->p2 / 16; out->tn = d->p2 / 16;
    } else {
        out->wm = d->p1; out->wn = d->p2; out->tm = d->p1 / frag; out->tn = d->p2 / frag;
    }
    out->k_waves = d->kw;
    out->threads = d->threads;
    out->split_k = d->splitK;
    out->lds_bytes = d->ldsBytes;
    out->band_rows = d->band;
    out->balanced_per_cu = d->sk;
    std::call_once(g_once, init_tables);
    out->available = (dtype == KS_F32 ? g_f32[kernel_id] : g_bf16[kernel_id]) != nullptr ? 1 : 0;
    return KS_OK;
}

extern "C" int ks_calibration_copy(void *dst, const void *src, size_t bytes, void *stream) {
    if (!dst || !src || bytes == 0 || bytes % 16 != 0) return KS_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(dst) % 16 || reinterpret_cast<uintptr_t>(src) % 16)
        return KS_ERR_INVALID_ARG;
    (void)hipGetLastError();
    const long long n16 = (long long)(bytes / 16);
    const int grid = (int)((n16 + 255) / 256 < 16384 ? (n16 + 255) / 256 : 16384);
    hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const floatx4 *>(src), static_cast<floatx4 *>(dst), n16);
    return hipGetLastError() == hipSuccess ? KS_OK : KS_ERR_LAUNCH;
}

extern "C" int ks_set_fast_path(int enabled) {
    g_forceGeneric = enabled ? 0 : 1;
    return KS_OK;
}

extern "C" int ks_set_tiles_per_workgroup(int n) {
    if (n < 0 || n > 64) return KS_ERR_INVALID_ARG;
    g_tilesPerWG = n;
    return KS_OK;
}

extern "C" int ks_set_balanced_groups(int per_cu) {
    if (per_cu < 0 || per_cu > 8) return KS_ERR_INVALID_ARG;
    g_skPerCU = per_cu;
    return KS_OK;
}

extern "C" int ks_set_tail_split(int partitions) {
    if (partitions != -1 && partitions != 0 && (partitions < 2 || partitions > 16)) return KS_ERR_INVALID_ARG;
    g_tailSplit = partitions;
    return KS_OK;
}

extern "C" int ks_set_operand_copies(int mode) {
    if (mode < -1 || mode > 1) return KS_ERR_INVALID_ARG;
    g_operandCopies = mode;
    return KS_OK;
}

extern "C" int ks_set_split_partitions(int partitions) {
    if (partitions < 0 || partitions > 256) return KS_ERR_INVALID_ARG;
    g_splitForced = partitions;
    return KS_OK;
}

extern "C" int ks_set_workspace(void *device_ptr, size_t bytes) {
    if (device_ptr == nullptr || bytes == 0) {
        g_ws = nullptr;
        g_wsBytes = 0;
        return KS_OK;
    }
    if (reinterpret_cast<uintptr_t>(device_ptr) % sizeof(float)) return KS_ERR_INVALID_ARG;
    g_ws = device_ptr;
    g_wsBytes = bytes;
    return KS_OK;
}

extern "C" size_t ks_workspace_bytes_needed(int dtype, int kernel_id, int64_t M, int64_t N,
                                            int64_t batch) {
    const InstanceDesc *d = desc_of(dtype, kernel_id);
    if (!d || M <= 0 || N <= 0 || batch <= 0) return 0;
    if (d->sk > 0) return sk_workspace_bytes(d);
    if (d->splitK == 1) return 0;
    int64_t s = d->splitK;
    if (s == 0) {
        const int64_t tiles = ((M + d->bm - 1) / d->bm) * ((N + d->bn - 1) / d->bn) * batch;
        s = auto_split_max(d, tiles, dtype == KS_F32);
        if (s <= 1) return dtype != KS_F32 && batch == 1 ? tail_split_bytes(d, tiles) : 0;
    }
    return (size_t)s * (size_t)batch * (size_t)M * (size_t)N * sizeof(float);
}

#define KS_GEMM_PASS                                                                            \
    transA, transB, M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, batch, strideA, strideB, strideC, \
        static_cast<hipStream_t>(stream)

// Kernel for the selecting entry points: the choice of ks_select, unless the scratch does not hold its partial sums.
// Where a rule counts on a K split (selector.cpp), it is left out when the scratch holds fewer partitions than the member
// takes by its estimate, which is what the rule was timed with.  For an instance with a fixed split the one with the
// same tiles and no split is used instead, so that a caller who never registers a workspace is still served.
static int select_checked(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int tA, int tB,
                          Workspace w = registered_ws()) {
    int id = ks::select_member(dtype, M, N, K, batch, tA, tB, true);
    if (id < 0) return id;
    const InstanceDesc *d = desc_of(dtype, id);
    const int unsplit = ks::split_decides(dtype, M, N, K, batch) ? ks::select_member(dtype, M, N, K, batch, tA, tB, false) : id;
    if (unsplit != id && d && d->splitK == 0 &&
        (!w.ptr || partitions(d, dtype == KS_F32, M, N, K, batch, w) <
                       partitions(d, dtype == KS_F32, M, N, K, batch, Workspace{w.ptr, SIZE_MAX}))) {
        id = unsplit;
        d = desc_of(dtype, id);
    }
    if (!d || d->splitK <= 1 || M <= 0 || N <= 0 || batch <= 0) return id;
    const size_t need = (size_t)d->splitK * (size_t)batch * (size_t)M * (size_t)N * sizeof(float);
    if (w.ptr && w.bytes >= need) return id;
    const int n = dtype == KS_F32 ? kNumF32 : kNumBf16;
    std::call_once(g_once, init_tables);
    for (int pass = 0; pass < 2; ++pass)          // same K-step first, then any K-step
        for (int i = 0; i < n; ++i) {
            const InstanceDesc *e = desc_of(dtype, i);
            if ((dtype == KS_F32 ? g_f32[i] : g_bf16[i]) != nullptr &&      // present in a pruned build
                e->splitK == 1 && e->core == d->core && e->bm == d->bm && e->bn == d->bn &&
                e->p1 == d->p1 && e->p2 == d->p2 && (pass == 1 || e->bk == d->bk))
                return i;
        }
    return id;
}

namespace ks {
namespace {
// member that runs the remainder of a K range that is not a whole number of K-steps (run_ws)
int remainder_member(int dtype, int64_t M, int64_t N, int64_t K, int64_t batch, int tA, int tB, Workspace w) {
    const int id = select_checked(dtype, M, N, K, batch, tA, tB, w);
    if (id < 0) return id;
    std::call_once(g_once, init_tables);
    return g_bf16[id] != nullptr ? id : -1;
}
}  // namespace
}  // namespace ks

extern "C" int ks_gemm_f32_with_kernel(int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                       int64_t K, float alpha, const float *A, int64_t lda,
                                       const float *B, int64_t ldb, float beta, float *C, int64_t ldc,
                                       int64_t batch, int64_t strideA, int64_t strideB,
                                       int64_t strideC, void *stream) {
    return run(KS_F32, kernel_id, KS_GEMM_PASS);
}

extern "C" int ks_gemm_bf16_with_kernel(int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                        int64_t K, float alpha, const uint16_t *A, int64_t lda,
                                        const uint16_t *B, int64_t ldb, float beta, float *C,
                                        int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                                        int64_t strideC, void *stream) {
    return run(KS_BF16, kernel_id, KS_GEMM_PASS);
}

extern "C" int ks_gemm_f32(int transA, int transB, int64_t M, int64_t N, int64_t K, float alpha,
                           const float *A, int64_t lda, const float *B, int64_t ldb, float beta,
                           float *C, int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                           int64_t strideC, void *stream) {
    const int id = select_checked(KS_F32, M, N, K, batch, transA, transB);
    if (id < 0) return id;
    return run(KS_F32, id, KS_GEMM_PASS);
}

extern "C" int ks_gemm_bf16(int transA, int transB, int64_t M, int64_t N, int64_t K, float alpha,
                            const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, float beta,
                            float *C, int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                            int64_t strideC, void *stream) {
    const int id = select_checked(KS_BF16, M, N, K, batch, transA, transB);
    if (id < 0) return id;
    return run(KS_BF16, id, KS_GEMM_PASS, nullptr, 0, true);
}

extern "C" int ks_gemm_f16(int transA, int transB, int64_t M, int64_t N, int64_t K, float alpha,
                           const uint16_t *A, int64_t lda, const uint16_t *B, int64_t ldb, float beta,
                           float *C, int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                           int64_t strideC, void *stream) {
    const int id = select_checked(KS_F16, M, N, K, batch, transA, transB);
    if (id < 0) return id;
    return run(KS_F16, id, KS_GEMM_PASS, nullptr, 0, true);
}

extern "C" int ks_gemm_f16_with_kernel(int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                       int64_t K, float alpha, const uint16_t *A, int64_t lda,
                                       const uint16_t *B, int64_t ldb, float beta, float *C,
                                       int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                                       int64_t strideC, void *stream) {
    return run(KS_F16, kernel_id, KS_GEMM_PASS);
}

extern "C" int ks_gemm_bias(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N,
                            int64_t K, float alpha, const void *A, int64_t lda, const void *B,
                            int64_t ldb, float beta, float *C, int64_t ldc, const float *bias,
                            int64_t batch, int64_t strideA, int64_t strideB, int64_t strideC,
                            void *stream) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB);
        if (kernel_id < 0) return kernel_id;
    }
    return run(dtype, kernel_id, KS_GEMM_PASS, bias, 0, selected);
}

extern "C" int ks_gemm_out_bf16(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                int64_t K, float alpha, const void *A, int64_t lda, const void *B,
                                int64_t ldb, float beta, uint16_t *C16, int64_t ldc, const float *bias,
                                int64_t batch, int64_t strideA, int64_t strideB, int64_t strideC,
                                void *stream) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB);
        if (kernel_id < 0) return kernel_id;
    }
    float *C = reinterpret_cast<float *>(C16);        // element size is carried by the out16 flag
    return run(dtype, kernel_id, KS_GEMM_PASS, bias, 1, selected);
}

// Entry point for callers that cannot allocate device memory (HIP graph capture, serving loops):
// split-K partial sums go to a static device array instead of a registered workspace.
#define KS_STATIC_SCRATCH_BYTES (16u << 20)
namespace ks {
namespace {
__device__ __align__(256) float scratch[KS_STATIC_SCRATCH_BYTES / sizeof(float)];
constexpr int kMaxDevices = 64;
float *g_scratchPtr[kMaxDevices];      // device address of `scratch` on each device, once known
std::mutex g_scratchMutex;

// Device address of this device's copy of the static array (every device holds its own).  The
// array's name is only a host-side handle: the address kernels can use comes from the runtime.
int static_scratch(Workspace *out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return KS_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratchMutex);
    if (!g_scratchPtr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return KS_ERR_LAUNCH;
        }
        g_scratchPtr[dev] = static_cast<float *>(ptr);
    }
    out->ptr = g_scratchPtr[dev];
    out->bytes = KS_STATIC_SCRATCH_BYTES;
    return KS_OK;
}
}  // namespace
}  // namespace ks

extern "C" int ks_gemm_static_scratch(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                      int64_t K, float alpha, const void *A, int64_t lda, const void *B,
                                      int64_t ldb, float beta, float *C, int64_t ldc, int64_t batch,
                                      int64_t strideA, int64_t strideB, int64_t strideC, void *stream) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    Workspace w{nullptr, 0};
    const int rc = static_scratch(&w);
    if (rc != KS_OK) return rc;
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB, w);
        if (kernel_id < 0) return kernel_id;
    }
    return run_ws(w, dtype, kernel_id, KS_GEMM_PASS, nullptr, 0, nullptr, false, false, selected);
}

extern "C" int ks_gemm_with_workspace(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N,
                                      int64_t K, float alpha, const void *A, int64_t lda, const void *B,
                                      int64_t ldb, float beta, float *C, int64_t ldc, int64_t batch,
                                      int64_t strideA, int64_t strideB, int64_t strideC, void *workspace_device,
                                      size_t workspace_bytes, void *stream) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    if ((workspace_device == nullptr) != (workspace_bytes == 0)) return KS_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace_device) % sizeof(float)) return KS_ERR_INVALID_ARG;
    const Workspace w{workspace_device, workspace_bytes};
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB, w);
        if (kernel_id < 0) return kernel_id;
    }
    return run_ws(w, dtype, kernel_id, KS_GEMM_PASS, nullptr, 0, nullptr, true, false, selected);
}

extern "C" int ks_gemm_plan(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N, int64_t K,
                            float alpha, const void *A, int64_t lda, const void *B, int64_t ldb, float beta,
                            float *C, int64_t ldc, int64_t batch, int64_t strideA, int64_t strideB,
                            int64_t strideC, ks_launch_plan_t *out) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    if (!out) return KS_ERR_INVALID_ARG;
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB);
        if (kernel_id < 0) return kernel_id;
    }
    void *stream = nullptr;
    return run_ws(registered_ws(), dtype, kernel_id, KS_GEMM_PASS, nullptr, 0, out, false, false, selected);
}

extern "C" int ks_time_gemm(int dtype, int kernel_id, int transA, int transB, int64_t M, int64_t N,
                            int64_t K, float alpha, const void *A, int64_t lda, const void *B,
                            int64_t ldb, float beta, float *C, int64_t ldc, int64_t batch,
                            int64_t strideA, int64_t strideB, int64_t strideC, void *stream,
                            int warmup, int iters, int reps, float *ms_out) {
    if (dtype != KS_F32 && dtype != KS_BF16 && dtype != KS_F16) return KS_ERR_INVALID_ARG;
    if (iters < 1 || iters > 1024 || reps < 1 || warmup < 0 || !ms_out) return KS_ERR_INVALID_ARG;
    const bool selected = kernel_id < 0;
    if (selected) {
        kernel_id = select_checked(dtype, M, N, K, batch, transA, transB);
        if (kernel_id < 0) return kernel_id;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // one pool of events per host thread (events are created once and reused by later calls)
    static thread_local hipEvent_t ev[2 * 1024];
    static thread_local int evCount = 0;
    while (evCount < 2 * iters) {
        if (hipEventCreate(&ev[evCount]) != hipSuccess) return KS_ERR_LAUNCH;
        ++evCount;
    }
    // the first launch also proves the arguments: if it is refused nothing else is enqueued
    int rc = KS_OK;
    for (int i = 0; i < warmup; ++i) {
        rc = run(dtype, kernel_id, KS_GEMM_PASS, nullptr, 0, selected);
        if (rc != KS_OK) return rc;
    }
    for (int i = 0; i < iters; ++i) {
        if (hipEventRecord(ev[2 * i], s) != hipSuccess) return KS_ERR_LAUNCH;
        for (int r = 0; r < reps; ++r) {
            rc = run(dtype, kernel_id, KS_GEMM_PASS, nullptr, 0, selected);
            if (rc != KS_OK) return rc;
        }
        if (hipEventRecord(ev[2 * i + 1], s) != hipSuccess) return KS_ERR_LAUNCH;
    }
    if (hipStreamSynchronize(s) != hipSuccess) return KS_ERR_LAUNCH;
    for (int i = 0; i < iters; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]) != hipSuccess) return KS_ERR_LAUNCH;
        ms_out[i] = ms / (float)reps;
    }
    return KS_OK;
}
