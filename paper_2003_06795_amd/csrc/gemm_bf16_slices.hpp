// 16-bit products with few output tiles and a long K: every wave of a work-group computes the whole BM x BN tile over its own
// part of K (paper Section II: the inner-product engine and the launch shape are the kernel's axes).
//
// With fewer tiles than compute units the other members cut K over work-groups, which takes a second launch to add the
// partitions up (4 us of calls that take 6 to 40), or leave the device to a chain of K-steps at memory latency behind a barrier
// each.  Here wave w of NW takes K-steps w, w + NW, ... of BK, so that the waves read neighbouring pieces of the same rows at
// the same time; each has a ring of STAGES K-steps in LDS of its own, filled by direct-to-LDS loads, and waits for nobody: no
// barrier before the sums of the waves meet in LDS and are added in wave order (the bits follow from the sizes and the tile, the
// tile from slices_tile: layout, strides, alignment and the member's partitions have a say in it).
// One work-group to a compute unit (120 to 144 KB of stages, 64 to 96 KB in flight).  Bound by what the unit's memory pipe
// takes, 0.95 to 1.05 us per 100 KB of operands from L2 and about 6 TB/s from memory.
// us, members as selected before -> here, operands rotated through three sets: 8192 x 16 x 8192 NN 34.7 -> 22.8, 2048 x 16 x 2048 NT 6.0 -> 3.4
// (launches of a graph), 4096 x 32 x 4096 NT 10.8 -> 7.7, 512 x 512 x 2048 NN 10.6 -> 6.7, 128 x 128 x 2048 NN 6.4 -> 4.1, 1024 x 1024 x 4096 NT 19.8 -> 19.4.
//
// An operand whose pieces one work-group each reads and that is large enough to be gone from the last-level cache before it is used
// again is loaded past it (NT_A, NT_B of `stream`): 8192 x 16 x 8192 26.6 -> 22.9 us, 14336 x 16 x 8192 46.8 -> 41.8 (5.6 TB/s); slices.hpp
// has the line and what it costs where nothing else comes in between.
// Preconditions are those of gemm_bf16_dma.hpp, K a multiple of 64, no K partitions over work-groups.
//
// gemm_bf16_slices_staged_kernel is the same for operands that nothing aligns: a wave holds PF K-steps in registers, as the members'
// register-staged path loads them (Bf16Staging), and passes them through one stage of its own (48 to 128 KB of LDS).  1000 x 777 x 1509 fp16 NN 17.6 -> 13.7 us;
// 1597 drawn products (64 .. 4096, skinny and tall, rows padded by up to three) of which 521 take it 0.70 of the time.
#pragma once
#include "gemm_bf16_dma.hpp"
#include "slices.hpp"

namespace ks {

enum { SLICES_NT_A = 1, SLICES_NT_B = 2 };

// One direct-to-LDS load, 16 bytes per lane from `from` bytes behind `tile` to lds + 16 * lane.  In asm as in
// gemm_bf16_pp.hpp: the compiler would wait for all loads in flight before it reads a stage, which it cannot tell from the one
// being filled.  M0 is written here and read by nothing else in the kernel; waits are explicit (wait_for_stage).
template <bool NT>
__device__ __forceinline__ void load_to_lds(unsigned from, const char *tile, char *lds) {
    const unsigned dst = (unsigned)(uintptr_t)(lds_void_ptr)lds;
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" : : "v"(from), "s"(tile), "s"(dst) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(from), "s"(tile), "s"(dst) : "memory");
}
// all but the N youngest loads have landed; no LDS read moves ahead of it
template <int N>
__device__ __forceinline__ void wait_for_stage() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// the LDS reads issued so far have returned; what they read may be overwritten
__device__ __forceinline__ void wait_for_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Lanes of a wave pass each other what they write to LDS: the LDS serves a wave's accesses in order, and the compiler, which sees the
// addresses of one lane only, keeps them in that order across this (no instruction).
__device__ __forceinline__ void lanes_meet() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

template <int BM, int BN, int BK, int NW, int STAGES, bool AKC, bool BKC, bool F16>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_slices_kernel(KS_PARAMS, const int stream) {
    KS_PARAMS_TOGETHER;
    constexpr int FM = BM / 16, FN = BN / 16, NF = FM * FN;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
    static_assert(NW * STAGES * STAGE <= 160 * 1024 && STAGES >= 2 && STAGES <= 4, "LDS");
    static_assert(NF * 1024 <= STAGES * STAGE, "a wave's sums in its own stages");
    __shared__ __attribute__((aligned(1024))) char lds[NW][STAGES][STAGE];
    using PlanA = DmaPlan<BM, BK, 1, AKC, 16>;
    using PlanB = DmaPlan<BN, BK, 1, BKC, 16>;
    constexpr int LOADS = PlanA::TOTAL + PlanB::TOTAL;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const TileCoord tc = tile_of_block(p);
    const int row0 = tc.tm * BM, col0 = tc.tn * BN;
    const uint16_t *Ab = static_cast<const uint16_t *>(p.A), *Bb = static_cast<const uint16_t *>(p.B);
    const int steps = p.K / BK, n = wave < steps ? (steps - wave + NW - 1) / NW : 0;      // this wave's K-steps
    const char *aTile = reinterpret_cast<const char *>(AKC ? Ab + (long long)row0 * p.lda + wave * BK : Ab + (long long)wave * BK * p.lda + row0);
    const char *bTile = reinterpret_cast<const char *>(BKC ? Bb + (long long)col0 * p.ldb + wave * BK : Bb + (long long)wave * BK * p.ldb + col0);
    const long long aStep = (AKC ? BK * 2LL : BK * 2LL * p.lda) * NW, bStep = (BKC ? BK * 2LL : BK * 2LL * p.ldb) * NW;

    PlanA pa;
    PlanB pb;
    pa.init(0, lane, p.lda, row0, AKC ? p.M : dma_extent(p.M));
    pb.init(0, lane, p.ldb, col0, BKC ? p.N : dma_extent(p.N));
    auto issue = [&](int t, int s) {
        char *const to = lds[wave][s];
        const char *const a = aTile + t * aStep, *const b = bTile + t * bStep;
        auto tile = [&](const auto &plan, const char *from, char *at, bool nt) {
            constexpr int TOTAL = std::remove_reference_t<decltype(plan)>::TOTAL;
            if (nt) {
#pragma unroll
                for (int j = 0; j < TOTAL; ++j) load_to_lds<true>(plan.off[j], from, at + j * 1024);
            } else {
#pragma unroll
                for (int j = 0; j < TOTAL; ++j) load_to_lds<false>(plan.off[j], from, at + j * 1024);
            }
        };
        tile(pa, a, to, (stream & SLICES_NT_A) != 0);
        tile(pb, b, to + A_BYTES, (stream & SLICES_NT_B) != 0);
    };
    floatx4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const char *from) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 32) {
            bf16x8 a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = read_fragment<16, BM, BK, AKC>(from, i * 16, kk, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = read_fragment<16, BN, BK, BKC>(from + A_BYTES, j * 16, kk, lane);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma_16x16x32<F16>(a[i], b[j], acc[i][j]);
        }
    };

    // Step t lives in stage t % STAGES.  Before it is read at most the loads of the younger steps are in flight; the stage that
    // step t - 1 left is refilled with step t + STAGES - 1 once its fragments are in registers.  (They are where the MFMAs of
    // step t - 1 stand in front of the refill, which nothing but the wait here makes the compiler do.)
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < n) issue(s, s);
    for (int t0 = 0; t0 < n; t0 += STAGES) {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            const int t = t0 + s;
            if (t >= n) break;
            const int younger = min(n - 1 - t, STAGES - 2);
            if (STAGES > 3 && younger >= 2) wait_for_stage<2 * LOADS>();
            else if (STAGES > 2 && younger >= 1) wait_for_stage<LOADS>();
            else wait_for_stage<0>();
            if (t + STAGES - 1 < n) {
                wait_for_reads();
                issue(t + STAGES - 1, (s + STAGES - 1) % STAGES);
            }
            multiply(lds[wave][s]);
        }
    }

    // the sums of a wave in its own stages, which it has read and nobody else writes
    floatx4 *const mine = reinterpret_cast<floatx4 *>(lds[wave][0]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) mine[(i * FN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += NW) {
        const int f = f0 + wave;
        if (f >= NF) break;
        floatx4 sum[1][1];
        sum[0][0] = reinterpret_cast<const floatx4 *>(lds[0][0])[f * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum[0][0] += reinterpret_cast<const floatx4 *>(lds[w][0])[f * 64 + lane];
        write_tile_mfma16<false, 1, 1>(p, tc, p.C, row0 + (f / FN) * 16, col0 + (f % FN) * 16, lane, sum);
    }
}

template <int BM, int BN, int BK, int NW, int PF, bool AKC, bool BKC, bool F16>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_slices_staged_kernel(const GemmParams p) {
    constexpr int FM = BM / 16, FN = BN / 16, NF = FM * FN;
    constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
    constexpr int OWN = STAGE > NF * 1024 ? STAGE : NF * 1024;       // a K-step, later the wave's sums
    static_assert(NW * OWN <= 160 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char lds[NW][OWN];
    using LoadA = Bf16Staging<BM, BK, 64, AKC, 16>;
    using LoadB = Bf16Staging<BN, BK, 64, BKC, 16>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const TileCoord tc = tile_of_block(p);
    const int row0 = tc.tm * BM, col0 = tc.tn * BN;
    const uint16_t *Ab = static_cast<const uint16_t *>(p.A), *Bb = static_cast<const uint16_t *>(p.B);
    // K-steps whose chunks may all be read whole (see Bf16Staging; rows of less than seven elements do not come here)
    const int fullA = AKC ? p.K / BK : (p.K - 1) / BK, fullB = BKC ? p.K / BK : (p.K - 1) / BK;
    const int full = min(fullA, fullB), steps = (p.K + BK - 1) / BK;
    const int n = wave < full ? (full - wave + NW - 1) / NW : 0;
    const long long aStep = (AKC ? (long long)BK : BK * p.lda) * NW, bStep = (BKC ? (long long)BK : BK * p.ldb) * NW;
    LoadA la;
    LoadB lb;
    la.init(Ab, p.lda, row0, p.M, wave * BK, lane);
    lb.init(Bb, p.ldb, col0, p.N, wave * BK, lane);
    uintx4 ra[PF][LoadA::PER], rb[PF][LoadB::PER];
    floatx4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    char *const as = lds[wave], *const bs = as + A_BYTES;
    auto multiply = [&]() {
#pragma unroll
        for (int kk = 0; kk < BK; kk += 32) {
            bf16x8 a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = read_fragment<16, BM, BK, AKC>(as, i * 16, kk, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = read_fragment<16, BN, BK, BKC>(bs, j * 16, kk, lane);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) acc[i][j] = mfma_16x16x32<F16>(a[i], b[j], acc[i][j]);
        }
    };
#pragma unroll
    for (int s = 0; s < PF; ++s)
        if (s < n) { la.load(ra[s], s * aStep, lane); lb.load(rb[s], s * bStep, lane); }
    for (int t0 = 0; t0 < n; t0 += PF) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            const int t = t0 + s;
            if (t >= n) break;
            lanes_meet();
            LoadA::store(ra[s], as, lane);
            LoadB::store(rb[s], bs, lane);
            lanes_meet();
            if (t + PF < n) { la.load(ra[s], (t + PF) * aStep, lane); lb.load(rb[s], (t + PF) * bStep, lane); }
            multiply();
        }
    }
    // the steps that hold the end of K, as a rule one, are dealt out after the whole ones
    for (int t = full + (wave - full % NW + NW) % NW; t < steps; t += NW) {
        const int k0 = t * BK;
        if ((AKC ? p.K : p.M) >= 8 && (BKC ? p.K : p.N) >= 8) {
            LoadA::load_edge_back(ra[0], Ab, p.lda, row0, p.M, k0, p.K, lane);
            LoadB::load_edge_back(rb[0], Bb, p.ldb, col0, p.N, k0, p.K, lane);
            LoadA::fit_edge(ra[0], row0, p.M, k0, p.K, lane);
            LoadB::fit_edge(rb[0], col0, p.N, k0, p.K, lane);
        } else {
            LoadA::load_edge(ra[0], Ab, p.lda, row0, p.M, k0, p.K, lane);
            LoadB::load_edge(rb[0], Bb, p.ldb, col0, p.N, k0, p.K, lane);
        }
        lanes_meet();
        LoadA::store(ra[0], as, lane);
        LoadB::store(rb[0], bs, lane);
        lanes_meet();
        multiply();
    }
    // the sums of the waves in wave order
    lanes_meet();
    floatx4 *const mine = reinterpret_cast<floatx4 *>(lds[wave]);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) mine[(i * FN + j) * 64 + lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += NW) {
        const int f = f0 + wave;
        if (f >= NF) break;
        floatx4 sum[1][1];
        sum[0][0] = reinterpret_cast<const floatx4 *>(lds[0])[f * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum[0][0] += reinterpret_cast<const floatx4 *>(lds[w])[f * 64 + lane];
        write_tile_mfma16<false, 1, 1>(p, tc, p.C, row0 + (f / FN) * 16, col0 + (f % FN) * 16, lane, sum);
    }
}

}  // namespace ks
