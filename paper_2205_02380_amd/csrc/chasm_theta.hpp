// chasm_theta.hpp -- kernels of the truncated-kernel evaluation of the Coulomb
// pseudo-differential operator Theta_V (Sec. 4, eq. 4.6 with the tensor of eq. 4.9).
//
// At one x the operator is a discrete convolution over the N_k^3 k-grid,
//   Theta(x, k_p) = sum_a z_a (2/pi^2) Im( e^{i phi_a.p} sum_p' T_{p-p'} e^{-i phi_a.p'} f_p' ),
//   phi_a,d = 2 (x_d - x_a,d) hk_d,
// which is 2 Re of the I+ term of eq. 4.2 (the I- term is minus its conjugate for real
// f; 2/(c_{3,1} i) with c_{3,1} = 2 pi^2).  As f is real, it is one convolution of f with
// the real odd kernel
//   H_q = sum_a z_a (2/pi^2) T_q sin(phi_a.q),
// so no modulated copy of f is needed: f is transformed once for all nuclei, and the
// spectrum of a real field is held by one of each pair of conjugate frequencies.
//
// Along k1 and k2 the convolution is a product after transforms of length P = 2 N_k of
// the zero-padded data.  The k1 frequencies are xi1 = m + 1/2, m < P (a skew-circular
// convolution: with N_k zeros behind N_k values it gives the same result as a circular
// one), so that conjugate pairs m, P - 1 - m are never one frequency and N_k of the P
// planes xi1 are held; the k2 frequencies are xi2 < P.  Along k3 it stays a product with a
// Toeplitz matrix.  With the even tensor T shifted in both frequencies,
//   K_a(xi1, xi2, q3) = sum_{q1, q2} T_q cos(phi_a,1 q1 - 2 pi xi1 q1 / P) cos(phi_a,2 q2 - 2 pi xi2 q2 / P),
//   D_a = K_a(xi1, xi2) - K_a(-xi1, -xi2),   S_a = K_a(xi1, xi2) + K_a(-xi1, -xi2),
// the transformed kernel is, up to weights,
//   sum_a S_a(q3) sin(phi_a,3 q3) - i D_a(q3) cos(phi_a,3 q3):
// an even and an odd real Toeplitz matrix per line (xi1, xi2).  D and S belong to a pair
// (x1, x2) of nodes and serve all x3 (and batch members): they are tables, 4 N_k^3 doubles
// per pair and nucleus, made by the kernels of chasm_theta_table.hpp.
//
// x-points are taken in the order t = (i1 nx2 + i2) nbatch nx3 + b nx3 + i3, in which the
// points of a pair are neighbours.  The one-block form of N_k = 8 and 16 is in
// chasm_theta_plane.hpp, the staged form in chasm_theta_big.hpp.
//
// The field is read and written in x-major order [b][x3][x2][x1][k3][k2][k1]; the
// transposes to and from the field layout are the kernels at the end of this file.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "chasm_fft.hpp"

namespace chasm {

constexpr int kMaxNuc = 4;

struct ThetaArgs {
    long long npts;              // x-points per batch member
    int nx[3];
    int nnuc, nbatch;
    double x_lo[3], hx[3], hk[3];
    double xa[kMaxNuc][3];       // nucleus positions
    double wgt[kMaxNuc];         // z_a (2/pi^2) / (2 P^2)
};

// The x-point of index t (see above): its line in the x-major field, its (x1, x2) pair and
// its x3 node.  There are fewer than 2^31 points.
struct XPoint {
    long long xp;
    unsigned pair;
    int i3;
};

__device__ __forceinline__ XPoint x_point(const ThetaArgs& a, unsigned t)
{
    const unsigned n3 = (unsigned)a.nx[2], m = n3 * (unsigned)a.nbatch;
    const unsigned pair = t / m, r = t % m, b = r / n3, i3 = r % n3;
    const unsigned i1 = pair / (unsigned)a.nx[1], i2 = pair % (unsigned)a.nx[1];
    return {b * a.npts + ((long long)i3 * a.nx[1] + i2) * a.nx[0] + i1, pair, (int)i3};
}

// Factors of a handle (k_theta_mod): 4 N_k values e^{-2 pi i n / (4 N_k)}, then for every
// nucleus the rows e^{-i phi k} (k < N_k) of the nx1 + nx2 + nx3 nodes of the three axes.
__host__ __device__ __forceinline__ const fft::cd* mod_row(const fft::cd* et, const ThetaArgs& a, int nk, int nu, int axis, int i)
{
    const int at = i + (axis > 0 ? a.nx[0] : 0) + (axis > 1 ? a.nx[1] : 0);
    return et + 4 * nk + ((long long)nu * (a.nx[0] + a.nx[1] + a.nx[2]) + at) * nk;
}

template <typename T, int NK>
__device__ __forceinline__ void load_k1(const T* __restrict__ p, double (&v)[NK])
{
    if constexpr (sizeof(T) == 4) {
        static_assert(NK % 4 == 0, "float4 rows");
        const float4* q = reinterpret_cast<const float4*>(p);
        fft::sfor<0, NK / 4>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const float4 t = q[i];
            v[4 * i] = t.x;
            v[4 * i + 1] = t.y;
            v[4 * i + 2] = t.z;
            v[4 * i + 3] = t.w;
        });
    } else {
        const double2* q = reinterpret_cast<const double2*>(p);
        fft::sfor<0, NK / 2>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const double2 t = q[i];
            v[2 * i] = t.x;
            v[2 * i + 1] = t.y;
        });
    }
}

// The same without the conversion.
template <typename T, int NK>
__device__ __forceinline__ void load_raw(const T* __restrict__ p, T (&v)[NK])
{
    using V = typename std::conditional<sizeof(T) == 4, float4, double2>::type;
    constexpr int n = sizeof(V) / sizeof(T);
    static_assert(NK % n == 0, "whole vectors");
    const V* q = reinterpret_cast<const V*>(p);
    fft::sfor<0, NK / n>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const V t = q[i];
        if constexpr (n == 4) {
            v[4 * i] = t.x;
            v[4 * i + 1] = t.y;
            v[4 * i + 2] = t.z;
            v[4 * i + 3] = t.w;
        } else {
            v[2 * i] = t.x;
            v[2 * i + 1] = t.y;
        }
    });
}

template <typename T, int NK>
__device__ __forceinline__ void store_k1(T* __restrict__ p, const double (&v)[NK])
{
    if constexpr (sizeof(T) == 4) {
        float4* q = reinterpret_cast<float4*>(p);
        fft::sfor<0, NK / 4>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            q[i] = make_float4((float)v[4 * i], (float)v[4 * i + 1], (float)v[4 * i + 2], (float)v[4 * i + 3]);
        });
    } else {
        double2* q = reinterpret_cast<double2*>(p);
        fft::sfor<0, NK / 2>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            q[i] = make_double2(v[2 * i], v[2 * i + 1]);
        });
    }
}

// out[b][c][r] = in[b][r][c] for an (rows x cols) matrix per batch member; 64 x 64
// tiles through LDS, 256 threads, coalesced on both sides.  The transposes of an LPC1
// step (Sec. 2.2) also form its combinations, which saves a pass over memory each:
//   TR_PREDICT  out = (in + c g) transposed         (g in the layout of in)
//   TR_CORRECT  out = out + c (g + in transposed)   (g in the layout of out)
enum TransposeMode { TR_PLAIN = 0, TR_PREDICT = 1, TR_CORRECT = 2 };

template <typename T, int MODE>
__global__ __launch_bounds__(256) void k_transpose(const T* __restrict__ in, const T* __restrict__ g, T* __restrict__ out,
                                                  long long rows, long long cols, T c)
{
    __shared__ T tile[64][65];
    const long long b = blockIdx.z;
    const long long r0 = (long long)blockIdx.y * 64, c0 = (long long)blockIdx.x * 64, base = b * rows * cols;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    for (int i = ty; i < 64; i += 4) {
        const long long r = r0 + i, cc = c0 + tx;
        if (r < rows && cc < cols) {
            const long long at = base + r * cols + cc;
            tile[i][tx] = MODE == TR_PREDICT ? fma(c, g[at], in[at]) : in[at];
        }
    }
    __syncthreads();
    for (int i = ty; i < 64; i += 4) {
        const long long cc = c0 + i, r = r0 + tx;
        if (r < rows && cc < cols) {
            const long long at = base + cc * rows + r;
            out[at] = MODE == TR_CORRECT ? fma(c, g[at] + tile[tx][i], out[at]) : tile[tx][i];
        }
    }
}

}  // namespace chasm
