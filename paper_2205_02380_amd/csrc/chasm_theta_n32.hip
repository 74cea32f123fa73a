// chasm_theta_n32.hip -- Theta_V kernels of the 32^3 k-grid.
#include "chasm_theta_launch.hpp"

namespace chasm {

static const ThetaKernels kKernels[2] = {
    {0, 32, nullptr, launch_transpose<float>, launch_big<float, 32>, launch_mod<32>, launch_node<32>, launch_table<32>},
    {1, 32, nullptr, launch_transpose<double>, launch_big<double, 32>, launch_mod<32>, launch_node<32>, launch_table<32>},
};

const ThetaKernels* theta_kernels_32() { return kKernels; }

}  // namespace chasm
