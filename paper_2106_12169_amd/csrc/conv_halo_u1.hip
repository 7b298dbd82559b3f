// Instances of conv_halo_kernel for features of one 0/1 plane.
#include "conv_halo_launch.h"

namespace apnn {

bool launch_conv_halo_u1(const ConvHaloParams &p, bool stay, int fp, unsigned grid, int lds, hipStream_t st)
{
    return launch_conv_halo<OPK_U1>(p, stay, fp, grid, lds, st);
}

}  // namespace apnn
