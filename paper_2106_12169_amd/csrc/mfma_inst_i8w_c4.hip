// Instances of the 8-bit integer matrix kernel with K shared out among the waves (mfma_i8_wide.h) whose row operand
// has plane class C4.
#include "common.h"
#include "mfma_i8_wide.h"
#include "mfma_launch.h"

namespace apnn {

template <int CB> static bool go(const MfmaParams &p, unsigned grid, hipStream_t st)
{
    auto kernel = mfma_i8_wide_kernel<I8_C4, CB>;
    const int lds = mfma_i8_wide_lds_bytes(p.PA, p.PB);
    static std::atomic<uint64_t> granted{0};
    if (!all_of_lds(kernel, granted)) return false;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), lds, st, p);
    return true;
}

bool launch_mfma_i8_wide_c4(const MfmaParams &p, int classB, unsigned grid, hipStream_t st)
{
    switch (classB) {
        case I8_C2: return go<I8_C2>(p, grid, st);
        case I8_C4: return go<I8_C4>(p, grid, st);
        case I8_C8: return go<I8_C8>(p, grid, st);
        default: return false;                           // (both operands above four planes: more LDS than there is)
    }
}

}  // namespace apnn
