// Instances of mfma_i8_kernel: every pair of plane classes.
#include "common.h"
#include "mfma_i8.h"
#include "mfma_launch.h"

namespace apnn {

template <int CA, int CB> static bool go(const MfmaParams &p, unsigned grid, hipStream_t st)
{
    const auto kernel = mfma_i8_kernel<CA, CB>;
    static std::atomic<uint64_t> granted{0};
    if (!all_of_lds(kernel, granted)) return false;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(512), kI8LdsBytes, st, p);
    return true;
}

bool launch_mfma_i8(const MfmaParams &p, int classA, int classB, unsigned grid, hipStream_t st)
{
    switch (3 * classA + classB) {
        case 0: return go<0, 0>(p, grid, st);
        case 1: return go<0, 1>(p, grid, st);
        case 2: return go<0, 2>(p, grid, st);
        case 3: return go<1, 0>(p, grid, st);
        case 4: return go<1, 1>(p, grid, st);
        case 5: return go<1, 2>(p, grid, st);
        case 6: return go<2, 0>(p, grid, st);
        case 7: return go<2, 1>(p, grid, st);
        case 8: return go<2, 2>(p, grid, st);
        default: return false;
    }
}

}  // namespace apnn
