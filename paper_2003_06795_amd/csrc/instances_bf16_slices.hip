// The K-slices form of the 16-bit products: every tile of slices.hpp in four layouts and both 16-bit types (in a pruned library too:
// no member names it).
#include "gemm_bf16_slices.hpp"

namespace ks {

template <int BM, int BN, int BK, int NW, int STAGES>
static void launch(const GemmParams &p, int grid, int variant, int stream, hipStream_t s) {
    const dim3 g = launch_grid(p, grid), b(64 * NW);
#define KS_V(A, B)                                                                                                            \
    do {                                                                                                                      \
        if (variant & 16) hipLaunchKernelGGL((gemm_bf16_slices_kernel<BM, BN, BK, NW, STAGES, A, B, true>), g, b, 0, s, KS_ARGUMENTS(p), stream); \
        else hipLaunchKernelGGL((gemm_bf16_slices_kernel<BM, BN, BK, NW, STAGES, A, B, false>), g, b, 0, s, KS_ARGUMENTS(p), stream);       \
    } while (0)
    switch (variant & 3) {
        case 0: KS_V(false, false); break;
        case 1: KS_V(false, true); break;
        case 2: KS_V(true, false); break;
        default: KS_V(true, true); break;
    }
#undef KS_V
}

template <int BM, int BN, int BK, int NW, int PF>
static void launch_staged(const GemmParams &p, int grid, int variant, hipStream_t s) {
    const dim3 g = launch_grid(p, grid), b(64 * NW);
#define KS_V(A, B)                                                                                                            \
    do {                                                                                                                      \
        if (variant & 16) hipLaunchKernelGGL((gemm_bf16_slices_staged_kernel<BM, BN, BK, NW, PF, A, B, true>), g, b, 0, s, p); \
        else hipLaunchKernelGGL((gemm_bf16_slices_staged_kernel<BM, BN, BK, NW, PF, A, B, false>), g, b, 0, s, p);            \
    } while (0)
    switch (variant & 3) {
        case 0: KS_V(false, false); break;
        case 1: KS_V(false, true); break;
        case 2: KS_V(true, false); break;
        default: KS_V(true, true); break;
    }
#undef KS_V
}

void launch_bf16_slices(int tile, const GemmParams &p, int grid, int variant, int stream, hipStream_t s) {
    switch (tile) {
#define KS_CASE(i, BM, BN, BK, NW, ST, FIXED) case i: launch<BM, BN, BK, NW, ST>(p, grid, variant, stream, s); break;
        KS_SLICES_TILES(KS_CASE)
#undef KS_CASE
#define KS_CASE(i, BM, BN, BK, NW, PF, FIXED) case i: launch_staged<BM, BN, BK, NW, PF>(p, grid, variant, s); break;
        KS_SLICES_STAGED_TILES(KS_CASE)
#undef KS_CASE
        default: break;
    }
}

}  // namespace ks
