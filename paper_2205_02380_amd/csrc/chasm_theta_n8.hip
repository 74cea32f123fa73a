// chasm_theta_n8.hip -- Theta_V kernels of the 8^3 k-grid.
#include "chasm_theta_launch.hpp"

namespace chasm {

static const ThetaKernels kKernels[2] = {
    {0, 8, launch_theta<float, 8>, launch_transpose<float>, nullptr, launch_mod<8>, launch_node<8>, launch_table<8>},
    {1, 8, launch_theta<double, 8>, launch_transpose<double>, nullptr, launch_mod<8>, launch_node<8>, launch_table<8>},
};

const ThetaKernels* theta_kernels_8() { return kKernels; }

}  // namespace chasm
