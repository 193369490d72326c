// 16-bit-input, fp32-accumulate members of the tiled GEMM family (paper Section II), MFMA only: the
// parts both operand paths share, and the register-staged path, which takes any operand.
//
// An instantiation fixes the work-group tile BM x BN, the K-step BK (multiple of 32), the wave
// tile WM x WN and the MFMA fragment F (32: v_mfma_f32_32x32x16_bf16, 16: v_mfma_f32_16x16x32_bf16).
//
// LDS layouts (both paths)
//   K-contiguous operand (A not transposed, B transposed):  tile[row][BK] in 16-byte chunks of eight
//     consecutive k; chunk c of row r sits at chunk position c ^ swz(r) (Bf16Lds), read with
//     ds_read_b128: the 16 lanes of one read phase, which want the same k-chunk of 16 consecutive
//     rows, fall into 16 different bank groups.
//   row-contiguous operand (A transposed, B not transposed): tile[k][ROWS] exactly as in memory;
//     32-byte units are XOR-swizzled by k (Bf16LdsT).  The MFMA operand (8 consecutive k of one row
//     per lane) is produced by the transposing LDS read ds_read_b64_tr_b16: inside each group of 16
//     lanes, lane s supplies the address of 4 consecutive rows at k = kb + s/4, and lane l
//     receives the 4 values k = kb .. kb+3 of row l.
//
//   AKC / BKC  operand is K-contiguous in memory (A: transA == 0, B: transB == 1)
#pragma once
#include <type_traits>

#include "ks_common.hpp"

namespace ks {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_void_ptr;

// The 16-bit members move bit patterns; only the MFMA instruction knows whether they are bf16 or
// IEEE binary16 (F16: v_mfma_f32_16x16x32_f16 / v_mfma_f32_32x32x16_f16).
template <bool F16>
__device__ __forceinline__ floatx4 mfma_16x16x32(bf16x8 a, bf16x8 b, floatx4 c) {
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
template <bool F16>
__device__ __forceinline__ floatx16 mfma_32x32x16(bf16x8 a, bf16x8 b, floatx16 c) {
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, a), __builtin_bit_cast(halfx8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <int BK>
struct Bf16Lds {
    static constexpr int CPR = BK / 8;            // 16-byte chunks per tile row
    static constexpr int RP = 16 / CPR;           // tile rows per 256 bytes of LDS
    static_assert(CPR == 4 || CPR == 8 || CPR == 16, "BK must be 32, 64 or 128");
    // index (in 16-byte units) of k-chunk c of tile row r
    __device__ __forceinline__ static int chunk(int r, int c) {
        return r * CPR + (c ^ ((r / RP) & (CPR - 1)));
    }
};

// F: fragment edge of the MFMAs that read the tile (the unit swizzle of narrow tiles depends on it)
template <int ROWS, int F = 32>
struct Bf16LdsT {
    static constexpr int CPR = ROWS / 8;                    // 16-byte chunks per k row
    static constexpr int UPR = ROWS / 16;                   // 32-byte units per k row
    // XOR applied to the 32-byte unit index of k row `k`.  A transposing read serves 32 lanes a pass, two groups of sixteen that
    // touch one unit each of four consecutive k rows: with 16 x 16 fragments the same unit of k and k + 8, with 32 x 32 ones
    // two neighbouring units, an even one and the next.  All eight have to land in different banks.  k rows of 256 bytes
    // and more start at the same one: two bits of k and bit 3, or the two bits above the one that tells the neighbours
    // apart.  Of 128 bytes, k and k + 1 differ by themselves and bit 1 of k (and bit 3) is left; of 64 bytes, four do.
    __device__ __forceinline__ static int swz(int k) {
        if constexpr (UPR >= 8) return F == 16 ? ((k & 3) | ((k >> 1) & 4)) : (k & 3) << 1;
        else if constexpr (UPR == 4) return F == 16 ? ((k & 2) | ((k >> 3) & 1)) : k & 2;
        else if constexpr (UPR == 2) return F == 16 ? ((k >> 3) & 1) : 0;
        else return 0;
    }
    // byte offset of element (k, row) for row a multiple of 4
    __device__ __forceinline__ static int byte_of(int k, int row) {
        return k * (ROWS * 2) + ((((row >> 4) ^ swz(k)) << 5) | ((row & 15) << 1));
    }
};

// LDS -> registers: the MFMA operand of one fragment, i.e. for lane l the eight consecutive k
// starting at kk + 8*(l / F) of tile row rowBase + l % F.  KC tiles ([row][BK], swizzled chunks)
// need one ds_read_b128; row-contiguous tiles ([k][ROWS]) two transposing ds_read_b64_tr_b16, in
// which lane s of a 16-lane group addresses rows 4*(s%4).. of k row s/4 and lane l receives the
// four k values of row l.
template <int F, int ROWS, int BK, bool KC>
__device__ __forceinline__ bf16x8 read_fragment(const char *tile, int rowBase, int kk, int lane) {
    const int lgrp = lane / F;
    if constexpr (KC) {
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4 *>(
            tile + 16 * Bf16Lds<BK>::chunk(rowBase + lane % F, kk / 8 + lgrp)));
    } else {
        typedef short shortx8 __attribute__((ext_vector_type(8)));
        using LT = Bf16LdsT<ROWS, F>;
        const int trRow = 4 * (lane & 3) + (F == 32 ? 16 * ((lane >> 4) & 1) : 0);
        shortx4 lo, hi;
        if constexpr (F == 32) {
            // The swizzle looks at bits 0 and 1 of k: k + 4 and the next k of a step are constants away.  One step from the LDS
            // array to the address: behind a chain of them the compiler no longer knows the array, takes the stage that
            // is read for the one being filled and waits for the loads in flight (64 x 64 x 64 NN 10.0 -> 11.8 us).
            int at = LT::byte_of(8 * lgrp + ((lane & 15) >> 2), rowBase + trRow);
            asm("" : "+v"(at));
            at += kk * (ROWS * 2);
            lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4 *)(lds_void_ptr)(tile + at));
            hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) shortx4 *)(lds_void_ptr)(tile + at + 4 * (ROWS * 2)));
        } else {
            // (the opaque offset costs 1024 x 4096 x 4096 TN on two groups of waves 1 %)
            const int kb = kk + 8 * lgrp + ((lane & 15) >> 2);
            lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) shortx4 *)(lds_void_ptr)(tile + LT::byte_of(kb, rowBase + trRow)));
            hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (__attribute__((address_space(3))) shortx4 *)(lds_void_ptr)(tile + LT::byte_of(kb + 4, rowBase + trRow)));
        }
        const shortx8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    }
}

// Scheduling hint for one k-substep: NM MFMAs with NR LDS reads spread evenly between them.
template <int M, int NM, int NR>
struct InterleaveHint {
    __device__ __forceinline__ static void emit() {
        if constexpr (M < NM) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // one MFMA
            // all reads go behind the first NM-2 MFMAs; the last two cover the read latency
            constexpr int SLOTS = NM > 2 ? NM - 2 : 1;
            constexpr int reads = M < SLOTS ? (NR * (M + 1)) / SLOTS - (NR * M) / SLOTS : 0;
            if constexpr (reads > 0) __builtin_amdgcn_sched_group_barrier(0x100, reads, 0);   // LDS reads
            InterleaveHint<M + 1, NM, NR>::emit();
        }
    }
};

// Global memory -> registers -> LDS for one operand tile of a K-step, ROWS x BK in the layout above.
// A thread moves the 16-byte chunks tid, tid + NT, ... of the LDS tile.
//
// load() is for K-steps in which every chunk may be read whole: the rows of a K-contiguous operand end
// at or behind the step, or the step of a row-contiguous one ends before the last k (a chunk that
// hangs over the right edge of row k then reads the beginning of row k + 1, and what it gets belongs to
// rows of C that do not exist).  Rows beyond `limit` are clamped to valid ones for the same reason.
// load_edge_back() / load_edge() are for the steps that are left, at most one for all but very narrow operands: they
// read inside the matrix only, and k beyond the end read as zero.
// load_units() serves any step of a K-contiguous operand whose K is a multiple of eight, with a test per chunk
// (the UNITS form of the kernel).
template <int ROWS, int BK, int NT, bool KC, int F>
struct Bf16Staging {
    static constexpr int CPR = (KC ? BK : ROWS) / 8;         // chunks along the contiguous direction
    static constexpr int CHUNKS = ROWS * BK / 8;
    static constexpr int PER = (CHUNKS + NT - 1) / NT;
    const uint16_t *src[PER];                                // this thread's chunks at the first K-step

    __device__ __forceinline__ static bool has(int tid, int j) { return CHUNKS % NT == 0 || tid + j * NT < CHUNKS; }

    __device__ __forceinline__ void init(const uint16_t *base, long long ld, int row0, int limit, int kBegin, int tid) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int L = tid + j * NT, outer = L / CPR, c = L % CPR;
            if constexpr (KC) {
                src[j] = base + (long long)min(row0 + outer, limit - 1) * ld + (kBegin + c * 8);
            } else {
                const int s = row0 + c * 8;
                src[j] = base + (long long)(kBegin + outer) * ld + (s < limit ? s : max(limit - 8, 0));
            }
        }
    }

    // advance: elements from the first K-step to this one
    __device__ __forceinline__ void load(uintx4 (&reg)[PER], long long advance, int tid) const {
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (has(tid, j)) reg[j] = load16_any(src[j] + advance);
    }

    // kLeft: k of the step that exist
    __device__ __forceinline__ void load_units(uintx4 (&reg)[PER], long long advance, int kLeft, int tid) const {
        static_assert(KC, "rows of a row-contiguous operand end anywhere");
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            uintx4 v = {0u, 0u, 0u, 0u};
            if (has(tid, j) && (tid + j * NT) % CPR * 8 < kLeft) v = load16_any(src[j] + advance);
            reg[j] = v;
        }
    }

    // load_edge() of an operand with at least eight elements along the contiguous direction: a chunk over the end is read
    // from further back, whole, and fit_edge() moves what exists of it to the front.  No branch, so the loads of a step wait
    // for memory once and not, chunk by chunk, for the elements of those over the end (every wave has some where the
    // operand is K-contiguous).  160 drawn calls on this path 0.94 of the time by this alone, 0.91 in NT, 0.95 in NN and TT, 0.96 in TN
    // (worst 1.05: 79 x 3010 x 151 TT): 1000 x 777 x 1509 NN 19.5 -> 17.9 us, 108 x 79 x 6085 NT in 39 partitions 8.5 -> 7.3; where few chunks
    // are over the end the moving shows (517 x 2936 x 152 TN 7.35 -> 7.6).
    __device__ __forceinline__ static void load_edge_back(uintx4 (&reg)[PER], const uint16_t *base, long long ld, int row0,
                                                          int limit, int k0, int kEnd, int tid) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int L = tid + j * NT, outer = L / CPR, c = L % CPR;
            const int line = KC ? min(row0 + outer, limit - 1) : min(k0 + outer, kEnd - 1);
            const int at = KC ? min(k0 + c * 8, kEnd - 8) : min(row0 + c * 8, limit - 8);
            if (has(tid, j)) reg[j] = load16_any(base + (long long)line * ld + at);
        }
    }
    __device__ __forceinline__ static void fit_edge(uintx4 (&reg)[PER], int row0, int limit, int k0, int kEnd, int tid) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int L = tid + j * NT, outer = L / CPR, c = L % CPR;
            if constexpr (!KC)
                if (row0 + ROWS <= limit) {               // no chunk of the tile hangs over
                    reg[j] = k0 + outer < kEnd ? reg[j] : uintx4{0u, 0u, 0u, 0u};
                    continue;
                }
            const int left = KC ? kEnd - (k0 + c * 8) : k0 + outer < kEnd ? limit - (row0 + c * 8) : 0;
            const int drop = 8 - max(0, min(left, 8)), b = 16 * (drop & 3);     // elements in front that are not the chunk's
            unsigned long long lo = reg[j][0] | (unsigned long long)reg[j][1] << 32;
            unsigned long long hi = reg[j][2] | (unsigned long long)reg[j][3] << 32;
            if (drop & 4) { lo = hi; hi = 0; }
            lo = lo >> b | (hi << 1) << (63 - b);
            hi >>= b;
            if (drop & 8) lo = hi = 0;
            reg[j] = uintx4{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
        }
    }

    __device__ __forceinline__ static void load_edge(uintx4 (&reg)[PER], const uint16_t *base, long long ld, int row0,
                                                     int limit, int k0, int kEnd, int tid) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const int L = tid + j * NT, outer = L / CPR, c = L % CPR;
            const int row = KC ? min(row0 + outer, limit - 1) : row0 + c * 8;
            const int k = KC ? k0 + c * 8 : k0 + outer;
            const int n = !has(tid, j) ? 0 : KC ? kEnd - k : k < kEnd ? limit - row : 0;   // elements that exist
            const uint16_t *p = KC ? base + (long long)row * ld + k : base + (long long)k * ld + row;
            uintx4 v = {0u, 0u, 0u, 0u};
            if (n >= 8) {
                v = load16_any(p);
            } else if (n > 0) {
                unsigned x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = p[min(e, n - 1)];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e >> 1] |= (e < n ? x[e] : 0u) << (16 * (e & 1));
            }
            reg[j] = v;
        }
    }

    __device__ __forceinline__ static void store(const uintx4 (&reg)[PER], char *lds, int tid) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (!has(tid, j)) continue;
            const int L = tid + j * NT, outer = L / CPR, c = L % CPR;
            const int at = KC ? Bf16Lds<BK>::chunk(outer, c) : outer * CPR + (c ^ (2 * Bf16LdsT<ROWS, F>::swz(outer)));
            reinterpret_cast<uintx4 *>(lds)[at] = reg[j];
        }
    }
};

// Register-staged path: operands whose rows are not 16-byte aligned, ragged extents and ragged K, in
// short everything the direct-to-LDS path does not take.  Same LDS tiles, same fragments, same order
// along K as that path, so on operands both take the results are the same bits.
//
// What bounds it is the latency of the operand loads: a K-step of most members holds 0.1 - 0.4 us of
// MFMAs against 1 - 2 us from memory.  Two K-steps are therefore in flight where two sets of staging
// registers of at most 32 fit beside at most 64 accumulators, one otherwise.  Measured against the
// element-wise loads (two bytes per lane, transposed in registers where row-contiguous) that this form
// replaced: fp16 1000 x 777 x 1509 NN 116 -> 19.6 us (17.9 since the last step reads back), bf16 5120 x 6528 x 2560 NT with odd rows 1312 ->
// 303 us (0.57 PFLOP/s), 4959 x 2007 x 1325 TN 713 -> 70 us.
//
// UNITS (both operands K-contiguous, K a multiple of eight): one loop of one kind of step, the next one in
// flight.  With one to three whole K-steps of 128 before a partial one the other form pays for the code of
// its unrolled loop and for a last step whose loads nothing hides: against the predicated sixteen-byte loads that
// aligned NT operands had before 64 x 16 tiles 1.08, with this form 1.03; 64 x 64 1.07 and 1.015; 128 x 128 on eight
// waves 1.05 and 1.02.  From four steps on, and with steps of 64 (1.02 at one whole step), the other one stays.
template <int F, int BM, int BN, int BK, int WM, int WN, bool SPLIT, bool AKC, bool BKC, bool F16 = false,
          bool UNITS = false>
__global__ __launch_bounds__(64 * (BM / WM) * (BN / WN)) void gemm_bf16_kernel(const GemmParams p) {
    constexpr int NT = 64 * (BM / WM) * (BN / WN);
    constexpr int FM = WM / F, FN = WN / F;
    constexpr int KSTEP = F == 32 ? 16 : 32;          // k consumed by one MFMA
    using LoadA = Bf16Staging<BM, BK, NT, AKC, F>;
    using LoadB = Bf16Staging<BN, BK, NT, BKC, F>;
    constexpr int PF = !UNITS && 4 * (LoadA::PER + LoadB::PER) <= 32 && WM * WN <= 4096 ? 2 : 1;
    __shared__ __attribute__((aligned(1024))) char As0[BM * BK * 2];
    __shared__ __attribute__((aligned(1024))) char As1[BM * BK * 2];
    __shared__ __attribute__((aligned(1024))) char Bs0[BN * BK * 2];
    __shared__ __attribute__((aligned(1024))) char Bs1[BN * BK * 2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const TileCoord tc = tile_of_block(p);
    const int row0 = tc.tm * BM, col0 = tc.tn * BN;
    const uint16_t *Ab = static_cast<const uint16_t *>(p.A) + (long long)tc.batch * p.strideA;
    const uint16_t *Bb = static_cast<const uint16_t *>(p.B) + (long long)tc.batch * p.strideB;
    float *Cb = p.C + (long long)tc.batch * p.strideC;
    const int kBegin = tc.split * p.kChunk;
    const int kEnd = min(p.K, kBegin + p.kChunk);
    const int nk = (kEnd - kBegin + BK - 1) / BK;
    const int subM = (wave / (BN / WN)) * WM, subN = (wave % (BN / WN)) * WN;

    // K-steps whose chunks may all be read whole (see Bf16Staging).  A row-contiguous operand with rows
    // of fewer than seven elements could reach beyond the row after next: it has none.
    const int fullA = AKC ? (kEnd - kBegin) / BK : p.lda < 7 ? 0 : (min(kEnd, p.K - 1) - kBegin) / BK;
    const int fullB = BKC ? (kEnd - kBegin) / BK : p.ldb < 7 ? 0 : (min(kEnd, p.K - 1) - kBegin) / BK;
    const int full = UNITS ? nk : max(min(fullA, fullB), 0);
    const long long aStep = AKC ? (long long)BK : BK * p.lda, bStep = BKC ? (long long)BK : BK * p.ldb;

    LoadA la;
    LoadB lb;
    la.init(Ab, p.lda, row0, p.M, kBegin, tid);
    lb.init(Bb, p.ldb, col0, p.N, kBegin, tid);
    uintx4 ra[PF][LoadA::PER], rb[PF][LoadB::PER];

    floatx4 acc16[F == 16 ? FM : 1][F == 16 ? FN : 1];
    floatx16 acc32[F == 32 ? FM : 1][F == 32 ? FN : 1];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
            if constexpr (F == 16) acc16[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
            else
#pragma unroll
                for (int e = 0; e < 16; ++e) acc32[i][j][e] = 0.f;
        }

    auto load = [&](int t, uintx4 (&a)[LoadA::PER], uintx4 (&b)[LoadB::PER]) {
        if constexpr (UNITS) {
            la.load_units(a, t * aStep, kEnd - kBegin - t * BK, tid);
            lb.load_units(b, t * bStep, kEnd - kBegin - t * BK, tid);
        } else {
            la.load(a, t * aStep, tid);
            lb.load(b, t * bStep, tid);
        }
    };
    // Wave tiles of 8192 entries and more read back where B is K-contiguous only: with both forms of the step beside their
    // accumulators, the unsplit 256 x 256 tile on 16-wide fragments spilled 48 registers instead of 39 in TN, inside its loop:
    // ragged calls without scratch for copies 1.06 of the time there (17, worst 1.15: 4981 x 1719 x 1551 73 -> 84 us), 1.00 (18, 1.06)
    // in NN against 0.99 without, 0.99 and 0.98 in NT and TT against 1.00.
    constexpr bool BACK = WM * WN < 8192 || BKC;
    // And only where a chunk can hang over an end: without one load_edge() reads each whole or not at all, and needs no moving
    // (80 calls on sizes of whole chunks with unaligned rows 0.98 of the time that reading back took, worst before 1.07 of the
    // form without it: 512 x 1656 x 152 TT, now 1.02; the remainders of a cut K 0.996).
    const int endA = AKC ? p.K : p.M, endB = BKC ? p.K : p.N;
    const bool back = BACK && (endA | endB) % 8 != 0 && endA >= 8 && endB >= 8;
    auto load_edge = [&](int t, uintx4 (&a)[LoadA::PER], uintx4 (&b)[LoadB::PER]) {
        const int k0 = kBegin + t * BK;
        if (back) {
            LoadA::load_edge_back(a, Ab, p.lda, row0, p.M, k0, kEnd, tid);
            LoadB::load_edge_back(b, Bb, p.ldb, col0, p.N, k0, kEnd, tid);
            LoadA::fit_edge(a, row0, p.M, k0, kEnd, tid);
            LoadB::fit_edge(b, col0, p.N, k0, kEnd, tid);
        } else {
            LoadA::load_edge(a, Ab, p.lda, row0, p.M, k0, kEnd, tid);
            LoadB::load_edge(b, Bb, p.ldb, col0, p.N, k0, kEnd, tid);
        }
    };
    auto compute = [&](const char *as, const char *bs) {
#pragma unroll
        for (int kk = 0; kk < BK; kk += KSTEP) {
            // large wave tiles have no registers for the fragments of two k-substeps at once
            if constexpr (WM * WN >= 8192) __builtin_amdgcn_sched_barrier(0);
            bf16x8 a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = read_fragment<F, BM, BK, AKC>(as, subM + i * F, kk, lane);
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = read_fragment<F, BN, BK, BKC>(bs, subN + j * F, kk, lane);
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    if constexpr (F == 16)
                        acc16[i][j] = mfma_16x16x32<F16>(a[i], b[j], acc16[i][j]);
                    else
                        acc32[i][j] = mfma_32x32x16<F16>(a[i], b[j], acc32[i][j]);
                }
        }
    };
    // K-step t sits in LDS stage t & 1 and came through register set t % PF; while it is consumed, that
    // set is refilled with step t + PF and step t + 1 moves from its set to the other stage.
    auto step = [&](int t, auto odd) {
        constexpr int S = decltype(odd)::value;
        constexpr int CUR = S % PF, NEXT = (S + 1) % PF;
        if (t + PF < full) load(t + PF, ra[CUR], rb[CUR]);
        compute(S ? As1 : As0, S ? Bs1 : Bs0);
        if (t + 1 < full) {
            LoadA::store(ra[NEXT], S ? As0 : As1, tid);
            LoadB::store(rb[NEXT], S ? Bs0 : Bs1, tid);
        }
        __syncthreads();
    };

    if constexpr (UNITS) {
        load(0, ra[0], rb[0]);
        LoadA::store(ra[0], As0, tid);
        LoadB::store(rb[0], Bs0, tid);
        __syncthreads();
        for (int t = 0; t < nk; ++t) {
            const bool odd = t & 1, more = t + 1 < nk;
            if (more) load(t + 1, ra[0], rb[0]);
            compute(odd ? As1 : As0, odd ? Bs1 : Bs0);
            if (more) {
                LoadA::store(ra[0], odd ? As0 : As1, tid);
                LoadB::store(rb[0], odd ? Bs0 : Bs1, tid);
            }
            __syncthreads();
        }
    } else if (full > 0) {
        load(0, ra[0], rb[0]);
        if (PF > 1 && full > 1) load(1, ra[PF - 1], rb[PF - 1]);
        LoadA::store(ra[0], As0, tid);
        LoadB::store(rb[0], Bs0, tid);
        __syncthreads();
        for (int t = 0; t < full; t += 2) {
            step(t, std::integral_constant<int, 0>{});
            if (t + 1 < full) step(t + 1, std::integral_constant<int, 1>{});
        }
    }
    // what is left: as a rule the one K-step that holds the end of K.  Every step above ended with a
    // barrier, so the first stage is free.
    for (int t = full; !UNITS && t < nk; ++t) {
        load_edge(t, ra[0], rb[0]);
        LoadA::store(ra[0], As0, tid);
        LoadB::store(rb[0], Bs0, tid);
        __syncthreads();
        compute(As0, Bs0);
        __syncthreads();
    }

    if constexpr (F == 16)
        write_tile_mfma16<SPLIT, FM, FN>(p, tc, Cb, row0 + subM, col0 + subN, lane, acc16);
    else
        write_tile_mfma32<SPLIT, FM, FN>(p, tc, Cb, row0 + subM, col0 + subN, lane, acc32);
}

}  // namespace ks
