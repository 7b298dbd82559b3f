// Instances of conv_halo_kernel for features of one -1/+1 plane.
#include "conv_halo_launch.h"

namespace apnn {

bool launch_conv_halo_pm1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st)
{
    return launch_conv_halo<OPK_PM1Z>(p, stay, fp, grid, lds, st);
}

}  // namespace apnn
