// chasm_theta_launch.hpp -- launchers of the Theta_V kernels.  The kernels of each k-grid
// size are instantiated in a unit of their own (chasm_theta_n<nk>.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_theta.hpp"
#include "chasm_theta_big.hpp"
#include "chasm_theta_plane.hpp"

namespace chasm {

// Compiled kernels: (storage type, nk) -> the one-block form (nk 8, 16) and the staged
// form over batches of x-points (nk 16, 32, 64).
using BigFn = hipError_t (*)(void* fx, const double* kt, const fft::cd* et, const ThetaArgs& a, fft::cd* W,
                             double* acc, long long total, long long X, hipStream_t s);

struct ThetaKernels {
    int dtype, nk;
    hipError_t (*theta)(void* fx, const double* kt, const fft::cd* et, const ThetaArgs& a, long long total,
                        hipStream_t s);
    hipError_t (*transpose)(int mode, const void* in, const void* g, void* out, long long rows, long long cols,
                            int batch, double c, hipStream_t s);
    BigFn big;                 // staged form (nullptr: none)
    hipError_t (*mod)(fft::cd* et, const ThetaArgs& a, hipStream_t s);
};

template <typename K>
long long resident(K k, int threads)
{
    int dev = 0, ncu = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, threads, 0) != hipSuccess) return 0;
    return (long long)ncu * (per > 0 ? per : 1);
}

template <typename T, int NK>
hipError_t launch_theta(void* fx, const double* kt, const fft::cd* et, const ThetaArgs& a, long long total,
                               hipStream_t s)
{
    auto k = k_theta<T, NK>;
    constexpr int NT = NK * NK;
    const long long res = resident(k, NT);
    const unsigned grid = (unsigned)(res > 0 && res < total ? res : total);
    hipLaunchKernelGGL(k, dim3(grid), dim3(NT), 0, s, static_cast<T*>(fx), kt, et, a, total);
    return hipGetLastError();
}

// The modulation table of a handle (k_theta_mod): rows of nk factors.
inline long long mod_rows(const ThetaArgs& a) { return 2 + (long long)a.nnuc * (a.nx[0] + a.nx[1] + a.nx[2]); }

template <int NK>
hipError_t launch_mod(fft::cd* et, const ThetaArgs& a, hipStream_t s)
{
    const long long n = NK * mod_rows(a);
    hipLaunchKernelGGL(k_theta_mod<NK>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, et, a);
    return hipGetLastError();
}

// Staged form: x-points in batches of X; per batch and nucleus the three stages.
template <typename T, int NK>
hipError_t launch_big(void* fx, const double* kt, const fft::cd* et, const ThetaArgs& a, fft::cd* W,
                             double* acc, long long total, long long X, hipStream_t s)
{
    using B = BigShape<NK>;
    for (long long x0 = 0; x0 < total; x0 += X) {
        const long long nb = total - x0 < X ? total - x0 : X;
        for (int nu = 0; nu < a.nnuc; ++nu) {
            hipLaunchKernelGGL((k_thA<T, NK>), dim3((unsigned)(nb * NK * NK / B::LA)), dim3(B::LA), 0, s,
                               static_cast<const T*>(fx), W, et, a, x0, nu);
            if constexpr (NK <= 32)
                hipLaunchKernelGGL((k_thBCD_plane<NK>), dim3((unsigned)(nb * B::P * 2 * NK / 64)), dim3(64), 0, s, W, kt,
                                   et, a, x0, nu);
            else
                hipLaunchKernelGGL((k_thBCD<NK>), dim3((unsigned)(nb * B::P)), dim3(B::NTB), 0, s, W, kt, et, a, x0, nu);
            hipLaunchKernelGGL((k_thE<T, NK>), dim3((unsigned)(nb * NK * NK / B::LE)), dim3(B::LE), 0, s, W, acc,
                               static_cast<T*>(fx), et, a, x0, nu, nu == 0 ? 1 : 0, nu == a.nnuc - 1 ? 1 : 0);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

template <typename T>
hipError_t launch_transpose(int mode, const void* in, const void* g, void* out, long long rows, long long cols, int batch,
                            double c, hipStream_t s)
{
    const dim3 grid((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64), (unsigned)batch);
    auto k = mode == TR_PLAIN ? k_transpose<T, TR_PLAIN> : mode == TR_PREDICT ? k_transpose<T, TR_PREDICT>
                                                                             : k_transpose<T, TR_CORRECT>;
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, static_cast<const T*>(in), static_cast<const T*>(g),
                       static_cast<T*>(out), rows, cols, (T)c);
    return hipGetLastError();
}

// The kernels of one nk for float and double fields.
const ThetaKernels* theta_kernels_8();
const ThetaKernels* theta_kernels_16();
const ThetaKernels* theta_kernels_32();
const ThetaKernels* theta_kernels_64();

}  // namespace chasm
