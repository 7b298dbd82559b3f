// Instances of the kernel for products and convolutions with few outputs: 16 x 16 tiles, K split over four or eight waves.
#include "mfma_launch.h"
#include "mfma_tile16.h"

namespace apnn {

template <int KA, int KB, int VW, bool CONV> static void go_vw(const MfmaParams &p, unsigned grid, hipStream_t st)
{
    hipLaunchKernelGGL((mfma_tile16_kernel<KA, KB, VW, CONV, 2>), dim3(grid), dim3(64 * p.nk), 0, st, p);
}

template <int KA, int KB> static bool go(const MfmaParams &p, int vw, unsigned grid, hipStream_t st)
{
    if (vw == 0) {
        if constexpr (KA == OPK_PM1Z) return false;
        else go_vw<KA, KB, 4, false>(p, grid, st);
    } else {
        if constexpr (KA == OPK_PM1) return false;      // (a convolution's -1/+1 features come with a validity word)
        else if (vw == 4) go_vw<KA, KB, 4, true>(p, grid, st);
        else if (vw == 2) go_vw<KA, KB, 2, true>(p, grid, st);
        else go_vw<KA, KB, 1, true>(p, grid, st);
    }
    return true;
}

bool launch_mfma_tile16(const MfmaParams &p, int kindA, int kindB, int vw, unsigned grid, hipStream_t st)
{
    switch (kindA * 3 + kindB) {
        case 0: return go<0, 0>(p, vw, grid, st);
        case 1: return go<0, 1>(p, vw, grid, st);
        case 2: return go<0, 2>(p, vw, grid, st);
        case 3: return go<1, 0>(p, vw, grid, st);
        case 4: return go<1, 1>(p, vw, grid, st);
        case 5: return go<1, 2>(p, vw, grid, st);
        case 6: return go<2, 0>(p, vw, grid, st);
        case 7: return go<2, 1>(p, vw, grid, st);
        case 8: return go<2, 2>(p, vw, grid, st);
        case 9: return go<3, 0>(p, vw, grid, st);
        case 10: return go<3, 1>(p, vw, grid, st);
        case 11: return go<3, 2>(p, vw, grid, st);
        default: return false;
    }
}

}  // namespace apnn
