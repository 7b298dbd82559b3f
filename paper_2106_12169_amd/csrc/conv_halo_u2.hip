// Instances of conv_halo_kernel for features of two-plane digits.
#include "conv_halo_launch.h"

namespace apnn {

bool launch_conv_halo_u2(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st)
{
    return launch_conv_halo<OPK_U2>(p, stay, fp, grid, lds, st);
}

}  // namespace apnn
