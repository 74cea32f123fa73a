// chasm_theta_n64.hip -- Theta_V kernels of the 64^3 k-grid.
#include "chasm_theta_launch.hpp"

namespace chasm {

static const ThetaKernels kKernels[2] = {
    {0, 64, nullptr, launch_transpose<float>, launch_big<float, 64>, launch_mod<64>, launch_node<64>, launch_table<64>},
    {1, 64, nullptr, launch_transpose<double>, launch_big<double, 64>, launch_mod<64>, launch_node<64>, launch_table<64>},
};

const ThetaKernels* theta_kernels_64() { return kKernels; }

}  // namespace chasm
