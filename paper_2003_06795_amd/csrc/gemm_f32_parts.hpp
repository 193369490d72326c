// fp32 members on the bf16 matrix pipe (paper Section II: the inner-product engine is one of the kernel's template axes).
//
// The matrix pipe multiplies bf16 sixteen times as fast as fp32.  A float is the sum of three bf16 numbers, x = h + m + l,
// each the rest of the one before rounded to nearest: 3 x 8 bits hold the 24 of the fraction.  The split is of 2^23 x: the last
// bit of any float is then 2^-126 or more and no part is a subnormal number (the matrix pipe keeps those, but a product of one
// loses its last bits), so that it is exact for every |x| up to 2^104, zero and subnormal ones too.  Accumulators hold
// 2^46 times the sum.
// Of the nine products of two such sums six are added: h h' into one fp32 accumulator, the small ones, h m', m h', m m', h l' and
// l h', into a second one, and the two into one another at the end.  |m| is up to 2^-8 and |l| up to 2^-17 of |x|: the three left
// out come to 2^-24 of a product at most.  An MFMA drops what lies about 24 bits below the largest of its sixteen products and of the
// accumulator: with the small products in an accumulator of their own that happens to a sum once in sixteen k, not six times.
// Error against fp64, rms over sum |a b|, fp32 pipe -> here, K = 49 / 128 / 2048 / 8192, 1e-8:
//   U[-1, 1) 2.4 / 2.4 / 2.4 / 2.4 -> 0.8 / 0.7 / 0.7 / 0.8      exp(2 N(0, 1)) 11 / 18 / 72 / 272 -> 6.3 / 8.0 / 25 / 49
//   U[0, 1) 10 / 16 / 60 / 119 -> 4.2 / 6.2 / 22 / 42             four terms of N(0, 1) 2.7 / 2.6 / 2.7 / 2.6 -> 1.9 / 1.9 / 1.9 / 1.9
//   one term 2.53 -> 2.59 at any K (at most 5.9 -> 9.2: the products left out); softmax(32 N(0, 1)) by N(0, 1), a few terms that are
//   nearly all of the sum, 3.2 / 3.6 / 4.4 / 4.6 -> 3.8 / 4.0 / 5.0 / 5.1.
// With all six in one accumulator U[-1, 1) comes to 2.0 / 1.9 / 2.0 / 2.2, four terms to 4.1 / 4.6 / 4.9 / 4.8, one term to 3.4.  Eight
// products bring one term to 2.53, for 1.07 of the time of two K groups, 1.15 on 64 x 64 tiles, 1.25 on 128 x 128 ones.
//
// What the accumulators cannot hold is computed on the fp32 matrix pipe, in the same launch: a work-group that ends with one that
// is no finite number (infinities and NaN of the operands, floats from 2^105 on, sums from 2^82 on) goes through its K range
// once more with fp32 tiles in the same LDS, and takes from it the entries that were not finite.  How an entry is computed depends
// on its row of A and its column of B alone, whatever the tile holds beside it.  Waves without such entries leave out
// the MFMAs: us, without -> one infinity / one in each tile: 4096^3 NT 633 -> 1024 / 1608, 2048^3 NN 103 -> 169 / 225,
// 480 x 1184 x 2592 TN 35.6 -> 53 / 52 (fp32 pipe 997, 165, 43).
//
// One K-step is 32 k whatever the member's: both operands' parts, 48 KB of a 128 x 128 tile, in one LDS stage of the 16-bit
// members' layouts (gemm_bf16.hpp); the next step's floats are in flight during the MFMAs and are split on their way to LDS.  Two
// work-groups of a compute unit fill each other's barriers, which takes eight waves in 128 registers: 64 of them are accumulators, so
// that parts live for a store only and a fragment of A for the products that it enters.  With two K groups, one or two
// work-groups to a unit, the floats are split behind the MFMAs (1600 x 982 x 3870 NN 102 -> 94 us, 480 x 1184 x 2592 TN 32.5 ->
// 31.6; 64 x 64 tiles with one group lose by it, 1000^3 NT 27.3 -> 29.6).  Bound by power on large problems (4096^3 at 215 TFLOP/s is
// 1.29 PFLOP/s of bf16) and by the sum of splitting (seven VALU instructions an element), LDS traffic and MFMAs on 64 x 64 tiles.
// Against the fp32 matrix pipe, us: 4096^3 NT 1000 -> 634, TN 1030 -> 672; 4095 x 3000 x 4089 NT 802 -> 529; 25088 x 256 x 1152 NN 140 -> 99;
// 2048^3 NN 150 -> 101; on 64 x 64 tiles 1944 x 1264 x 1576 TT 89 -> 67, 1000^3 NT 33.8 -> 28.0, with two K groups 480 x 1184 x 2592 TN
// 39.5 -> 31.8.
// Measured and left, with two accumulators: 64 x 64 of output per wave in 256 registers (1.2 to 1.4 of the time); one work-group of
// eight waves a unit, two LDS stages, one half of the waves splitting while the other multiplies (1.1 to 1.3); splitting
// behind the MFMAs on 128 x 128 tiles (128 registers do not hold the parts too: spills, 1.2 to 1.6); the sum of a K-step in
// registers of its own, added by VALU (1.5 to 2.3).  With one: two K-steps in flight (level to +4 %); v_dot2_f32_bf16 for the two steps of a rest
// (+5 to +12 %, and its inline -1.0 is the fp32 pattern); without s_setprio around the MFMAs +4 %.
#pragma once
#include "gemm_bf16.hpp"
#include "gemm_f32.hpp"

namespace ks {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// what the operands are multiplied by: the last bit of the smallest float, 2^-149, becomes 2^-126
constexpr float kPartsScale = 8388608.f;

// the parts of four floats, two to a register
struct FourParts {
    uintx2 part[3];
};
__device__ __forceinline__ FourParts split_parts(floatx4 x) {
    FourParts out;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        floatx2 v = {x[2 * h] * kPartsScale, x[2 * h + 1] * kPartsScale};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));      // to nearest, ties to even
            out.part[s][h] = u;
            if (s < 2) {
                v[0] -= __builtin_bit_cast(float, u << 16);
                v[1] -= __builtin_bit_cast(float, u & 0xFFFF0000u);
            }
        }
    }
    return out;
}

// The member's work-groups, tiles, waves, K groups, K ranges and accumulator layout (32x32 fragments) are those of
// gemm_f32_kernel, which describes SPLIT, KW and SK; only how a work-group multiplies a K range differs.
template <int BM, int BN, int P1, int P2, bool SPLIT, bool AKC, bool BKC, int KW, bool SK>
__global__ __launch_bounds__(64 * (BM / P1) * (BN / P2) * KW, 4) void gemm_f32_parts_kernel(const GemmParams p) {
    static_assert(!SK || (KW == 1 && !SPLIT), "balanced persistent form");
    constexpr int BK = 32, NT = 64 * (BM / P1) * (BN / P2), FM = P1 / 32, FN = P2 / 32;
    using KCA = std::integral_constant<bool, AKC>;
    using KCB = std::integral_constant<bool, BKC>;
    using LoaderA = TileLoader<BM, BK, NT, AKC, 4, AKC>;
    using LoaderB = TileLoader<BN, BK, NT, BKC, 4, BKC>;
    constexpr int PLANE_A = BM * BK * 2, PLANE_B = BN * BK * 2;
    constexpr int BYTES = 3 * (PLANE_A + PLANE_B);
    static_assert(4 * (LoaderA::LDS_SIZE + LoaderB::LDS_SIZE) <= BYTES, "fp32 tiles of a range computed again");
    static_assert(KW == 1 || BM * BN * 4 <= BYTES, "accumulators of the K groups");
    __shared__ __attribute__((aligned(1024))) char ldsAll[KW][BYTES];
    __shared__ int again;

    const int grp = KW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    char *const lds = ldsAll[grp];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x % NT >> 6);
    // (counted where it is needed: the balanced form's loop over tiles would keep it, and what follows from it, in registers)
    auto this_lane = []() {
        int zero = 0;
        asm volatile("" : "+v"(zero));
        return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, (unsigned)zero)) & 63;
    };
    const int subM = (wave / (BN / P2)) * P1, subN = (wave % (BN / P2)) * P2;
    floatx16 acc[FM][FN], low[FM][FN];                       // sums of h h', of the small products
    auto each = [&](auto f) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) f(i, j, e);
    };

    // acc = the products of k in [kLo, kHi) of the tile at (row, col), this group's slice of them
    auto range = [&](const float *A, const float *B, int row, int col, int kLo, int kHi) {
        const int lane = SK ? this_lane() : (int)threadIdx.x & 63, tid = SK ? wave * 64 + lane : (int)threadIdx.x % NT;
        const int nk = (max(kHi - kLo, 0) + KW * BK - 1) / (KW * BK);        // steps of the longest slice, for all groups
        const int kB = kLo + grp * nk * BK, kE = min(kHi, kB + nk * BK);     // kE may lie below kB: an empty slice
        typename LoaderA::Plan pa;
        typename LoaderB::Plan pb;
        pa.init(p.lda, row, p.M, tid);
        pb.init(p.ldb, col, p.N, tid);
        const int full = min(LoaderA::whole_steps(p.lda, p.M, p.K, kB, kE), LoaderB::whole_steps(p.ldb, p.N, p.K, kB, kE));
        LoaderA la;
        LoaderB lb;
        auto load = [&](int t) {
            const int k0 = kB + t * BK;
            if (t < full) {
                // (so that the compiler extends the offsets here and not, to two registers each, outside the K loop)
#pragma unroll
                for (unsigned &o : pa.off) asm volatile("" : "+v"(o));
#pragma unroll
                for (unsigned &o : pb.off) asm volatile("" : "+v"(o));
                la.load(pa, AKC ? A + (long long)row * p.lda + k0 : A + (long long)k0 * p.lda + row, p.lda, tid);
                lb.load(pb, BKC ? B + (long long)col * p.ldb + k0 : B + (long long)k0 * p.ldb + col, p.ldb, tid);
            } else {
                la.clear();
                lb.clear();
                la.load_edge(A, p.lda, row, p.M, k0, kE, tid);
                lb.load_edge(B, p.ldb, col, p.N, k0, kE, tid);
            }
        };
        // two K groups have the registers for a step's parts beside the MFMAs and split behind them
        constexpr bool BEHIND = KW == 2;
        FourParts ya[LoaderA::ITERS], yb[LoaderB::ITERS];
        auto split = [&]() {
            if constexpr (BEHIND) {
#pragma unroll
                for (int it = 0; it < LoaderA::ITERS; ++it) ya[it] = split_parts(la.reg[it]);
#pragma unroll
                for (int it = 0; it < LoaderB::ITERS; ++it) yb[it] = split_parts(lb.reg[it]);
            }
        };
        auto store = [&](auto rows, auto kc, char *to, const auto &l, const auto &behind) {
            constexpr int ROWS = decltype(rows)::value;
            constexpr bool KC = decltype(kc)::value;
            using L = TileLoader<ROWS, BK, NT, KC, 4, KC>;
            int from = tid;
            if constexpr (SK) {                              // (addresses that are made anew take no registers during the MFMAs)
                asm volatile("" : "+v"(from));
                from &= NT - 1;
            }
#pragma unroll
            for (int it = 0; it < L::ITERS; ++it) {
                const int inner = from % L::INNER, outer = from / L::INNER + it * L::STRIDE;
                const int at = KC ? 16 * Bf16Lds<BK>::chunk(outer, inner / 2) + 8 * (inner & 1)
                                  : Bf16LdsT<ROWS, 32>::byte_of(outer, inner * 4);
                const FourParts y = BEHIND ? behind[it] : split_parts(l.reg[it]);
#pragma unroll
                for (int s = 0; s < 3; ++s) *reinterpret_cast<uintx2 *>(to + s * (ROWS * BK * 2) + at) = y.part[s];
            }
        };
        auto multiply = [&](const char *from) {
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int kk = 0; kk < BK; kk += 16) {
                bf16x8 a[FM], b[FN], b1[FN];                 // one part of A at a time; one of B and its second
                auto readA = [&](int s) {
#pragma unroll
                    for (int i = 0; i < FM; ++i) a[i] = read_fragment<32, BM, BK, AKC>(from + s * PLANE_A, subM + i * 32, kk, lane);
                };
                auto readB = [&](bf16x8 (&b)[FN], int s) {
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        b[j] = read_fragment<32, BN, BK, BKC>(from + 3 * PLANE_A + s * PLANE_B, subN + j * 32, kk, lane);
                };
                auto mul = [&](floatx16 (&to)[FM][FN], bf16x8 (&b)[FN]) {
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j) to[i][j] = mfma_32x32x16<false>(a[i], b[j], to[i][j]);
                };
                readB(b, 0);
                readA(2);
                mul(low, b);
                readB(b1, 1);
                readA(1);
                mul(low, b1);
                mul(low, b);
                readA(0);
                mul(acc, b);
                mul(low, b1);
                readB(b, 2);
                mul(low, b);
            }
            __builtin_amdgcn_s_setprio(0);
        };
        each([&](int i, int j, int e) { acc[i][j][e] = low[i][j][e] = 0.f; });
        if (nk > 0) load(0);
        if (grp == 0 && tid == 0) again = 0;
        if (nk > 0) split();
        for (int t = 0; t < nk; ++t) {
            store(std::integral_constant<int, BM>{}, KCA{}, lds, la, ya);
            store(std::integral_constant<int, BN>{}, KCB{}, lds + 3 * PLANE_A, lb, yb);
            if (t + 1 < nk) load(t + 1);
            __syncthreads();
            multiply(lds);
            if (t + 1 < nk) split();
            __syncthreads();
        }
        float zero = 0.f;                                    // stays zero while the accumulators are finite
        each([&](int i, int j, int e) {
            acc[i][j][e] += low[i][j][e];
            zero = fmaf(acc[i][j][e], 0.f, zero);
            acc[i][j][e] *= 1.f / (kPartsScale * kPartsScale);
        });
        // (what the loads of a row-contiguous operand reach beyond its edge is none of the matrix's, whatever it holds)
        unsigned lost[FM][FN] = {};                          // bit e: accumulator e of the fragment
        if (!(zero == 0.f)) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    const int rows = p.M - (row + subM + i * 32 + 4 * (lane >> 5)), cols = p.N - (col + subN + j * 32 + (lane & 31));
                    unsigned bits = 0;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        bits |= !__builtin_isfinite(acc[i][j][e]) && 8 * (e / 4) + e % 4 < rows && cols > 0 ? 1u << e : 0u;
                    lost[i][j] = bits;
                    if (bits) again = 1;
                }
        }
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(again) != 0) {
            unsigned some = 0;
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) some |= lost[i][j];
            const bool mine = __any((int)some);
            each([&](int i, int j, int e) { low[i][j][e] = 0.f; });
            float *as = reinterpret_cast<float *>(lds), *bs = as + LoaderA::LDS_SIZE;
            load(0);
            for (int t = 0; t < nk; ++t) {
                la.store(as, tid);
                lb.store(bs, tid);
                if (t + 1 < nk) load(t + 1);
                __syncthreads();
                if (mine) {
#pragma unroll 1
                    for (int kk = 0; kk < BK; kk += 8) {
                        floatx4 a[FM], b[FN];
#pragma unroll
                        for (int i = 0; i < FM; ++i) a[i] = LoaderA::read(as, subM + i * 32 + (lane & 31), kk + 4 * (lane >> 5));
#pragma unroll
                        for (int j = 0; j < FN; ++j) b[j] = LoaderB::read(bs, subN + j * 32 + (lane & 31), kk + 4 * (lane >> 5));
#pragma unroll
                        for (int e = 0; e < 4; ++e)
#pragma unroll
                            for (int i = 0; i < FM; ++i)
#pragma unroll
                                for (int j = 0; j < FN; ++j)
                                    low[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], low[i][j], 0, 0, 0);
                    }
                }
                __syncthreads();
            }
            each([&](int i, int j, int e) {
                acc[i][j][e] = (lost[i][j] >> e) & 1u ? low[i][j][e] : acc[i][j][e];
            });
        }
        __syncthreads();                                     // LDS and `again` are the next range's
    };

    if constexpr (SK) {
        sk_for_each_tile<BK>(p, [&](const TileCoord &tc, int ks0, int ks1, int nkT, unsigned group, bool head) {
            const int row = tc.tm * BM, col = tc.tn * BN;
            range(static_cast<const float *>(p.A) + (long long)tc.batch * p.strideA,
                  static_cast<const float *>(p.B) + (long long)tc.batch * p.strideB, row, col, ks0 * BK, min(p.K, ks1 * BK));
            const int laneE = this_lane();
            if (ks0 == 0 && ks1 == nkT)
                write_tile_mfma32<false, FM, FN>(p, tc, p.C + (long long)tc.batch * p.strideC, row + subM, col + subN, laneE, acc);
            else
                sk_store_part<BM, BN, FM, FN>(p, group, head, wave, laneE, acc);
        });
    } else {
        const TileCoord tc = tile_of_block(p);
        const int row = __builtin_amdgcn_readfirstlane(tc.tm) * BM, col = __builtin_amdgcn_readfirstlane(tc.tn) * BN;
        const int kLo = tc.split * p.kChunk;
        range(static_cast<const float *>(p.A) + (long long)tc.batch * p.strideA,
              static_cast<const float *>(p.B) + (long long)tc.batch * p.strideB, row, col, kLo, min(p.K, kLo + p.kChunk));
        float *Cb = p.C + (long long)tc.batch * p.strideC;
        if constexpr (KW == 1) {
            write_tile_mfma32<SPLIT, FM, FN>(p, tc, Cb, row + subM, col + subN, (int)threadIdx.x & 63, acc);
        } else {
            constexpr int UNITS = (NT / 64) * FM * FN * 4 * 64;
            floatx4 *part = reinterpret_cast<floatx4 *>(ldsAll);
            store_units32<FM, FN>(part + grp * UNITS, wave, (int)threadIdx.x & 63, acc);
            __syncthreads();
            store_sum_of_groups<SPLIT, 32, 4, FM, FN, P1, P2, BN, NT, KW>(part, p, tc, Cb, row, col);
        }
    }
}

}  // namespace ks
