// chasm_theta_n16.hip -- Theta_V kernels of the 16^3 k-grid.
#include "chasm_theta_launch.hpp"

namespace chasm {

static const ThetaKernels kKernels[2] = {
    {0, 16, launch_theta<float, 16>, launch_transpose<float>, launch_big<float, 16>, launch_mod<16>, launch_node<16>, launch_table<16>},
    {1, 16, launch_theta<double, 16>, launch_transpose<double>, launch_big<double, 16>, launch_mod<16>, launch_node<16>, launch_table<16>},
};

const ThetaKernels* theta_kernels_16() { return kKernels; }

}  // namespace chasm
