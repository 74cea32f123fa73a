// chasm_theta_launch.hpp -- launchers of the Theta_V kernels.  The kernels of each k-grid
// size are instantiated in a unit of their own (chasm_theta_n<nk>.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_theta.hpp"
#include "chasm_theta_big.hpp"
#include "chasm_theta_plane.hpp"
#include "chasm_theta_table.hpp"

namespace chasm {

// x-points t0 .. t0 + n of a handle, and the range of its tables: pairs p0 .. p0 + np.
struct ThetaRange {
    long long t0, n;
    int p0, np;
};

// Compiled kernels: (storage type, nk) -> the one-block form (nk 8, 16) and the staged
// form (nk 16, 32, 64) on a range of x-points, and the tables of a range of pairs.
struct ThetaKernels {
    int dtype, nk;
    hipError_t (*theta)(void* fx, const double* tab, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r,
                        hipStream_t s);
    hipError_t (*transpose)(int mode, const void* in, const void* g, void* out, long long rows, long long cols,
                            int batch, double c, hipStream_t s);
    hipError_t (*big)(void* fx, const double* tab, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r, fft::cd* W,
                      hipStream_t s);   // nullptr: none
    hipError_t (*mod)(fft::cd* et, const ThetaArgs& a, hipStream_t s);
    hipError_t (*node)(double* U, const double* T, const fft::cd* et, const ThetaArgs& a, int i1_0, int n1, hipStream_t s);
    hipError_t (*table)(double* tab, const double* U, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r, int i1_0,
                        hipStream_t s);
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
hipError_t launch_theta(void* fx, const double* tab, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r,
                        hipStream_t s)
{
    auto k = k_theta<T, NK>;
    constexpr int NT = NK * NK;
    const long long res = resident(k, NT) / 8 * 8;
    const unsigned grid = (unsigned)(res > 0 && res < r.n ? res : r.n);
    hipLaunchKernelGGL(k, dim3(grid), dim3(NT), 0, s, static_cast<T*>(fx), tab, et, a, (unsigned)r.t0, (unsigned)r.n,
                       (unsigned)r.p0);
    return hipGetLastError();
}

// The factors of a handle (k_theta_mod): rows of nk.
inline long long mod_rows(const ThetaArgs& a) { return 4 + (long long)a.nnuc * (a.nx[0] + a.nx[1] + a.nx[2]); }

template <int NK>
hipError_t launch_mod(fft::cd* et, const ThetaArgs& a, hipStream_t s)
{
    const long long n = NK * mod_rows(a);
    hipLaunchKernelGGL(k_theta_mod<NK>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, et, a);
    return hipGetLastError();
}

// U of the nodes i1_0 .. i1_0 + n1, and the tables of a range from U of the nodes i1_0 ..
template <int NK>
hipError_t launch_node(double* U, const double* T, const fft::cd* et, const ThetaArgs& a, int i1_0, int n1, hipStream_t s)
{
    hipLaunchKernelGGL(k_theta_u<NK>, dim3((unsigned)n1 * a.nnuc, 2 * NK / 4), dim3(256), 0, s, U, T, et, a, i1_0);
    return hipGetLastError();
}

template <int NK>
hipError_t launch_table(double* tab, const double* U, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r, int i1_0,
                        hipStream_t s)
{
    hipLaunchKernelGGL(k_theta_table<NK>, dim3((unsigned)r.np * a.nnuc, NK / 4), dim3(256), 0, s, tab, U, et, a, r.p0, i1_0,
                       NK < 32 ? NK : 32);
    return hipGetLastError();
}

template <typename T, int NK>
hipError_t launch_big(void* fx, const double* tab, const fft::cd* et, const ThetaArgs& a, const ThetaRange& r, fft::cd* W,
                      hipStream_t s)
{
    using B = BigShape<NK>;
    const unsigned t0 = (unsigned)r.t0, p0 = (unsigned)r.p0, planes = (unsigned)(r.n * NK);
    hipLaunchKernelGGL((k_thA<T, NK>), dim3((unsigned)(r.n * NK * NK / B::LA)), dim3(B::LA), 0, s,
                       static_cast<const T*>(fx), W, a, t0);
    if constexpr (NK <= 32)
        hipLaunchKernelGGL((k_thBCD_plane<NK>), dim3(planes * 2 * NK / 64), dim3(64), 0, s, W, tab, et, a, t0, p0);
    else
        hipLaunchKernelGGL((k_thBCD<NK>), dim3(planes), dim3(B::NTB), 0, s, W, tab, et, a, t0, p0);
    hipLaunchKernelGGL((k_thE<T, NK>), dim3((unsigned)(r.n * NK * NK / B::LE)), dim3(B::LE), 0, s, W,
                       static_cast<T*>(fx), a, t0);
    return hipGetLastError();
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
