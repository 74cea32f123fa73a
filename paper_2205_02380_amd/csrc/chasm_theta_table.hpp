// chasm_theta_table.hpp -- the kernel tables D and S of Theta_V (notation as in
// chasm_theta.hpp): the factors of a grid's nodes, and for a range of (x1, x2) pairs
//   U[i1][nu][m][q2][q3] = w_nu sum_{q1} T_q cos(phi_1 q1 - 2 pi (m + 1/2) q1 / P),  m < P,
//   tab[pair][nu][c][D | S][q3 / 2][lane of xi2][q3 % 2],  c < N_k the held plane of
//   m = c / L + (P / L) (c % L).
// The lane of xi2 = 2 f + h is N_k h + f: the wave that works on a plane reads runs of 16
// N_k bytes (with q3 fastest every lane of a load touched a cache line of its own;
// with the loads also ahead of the row's transform, k_thBCD_plane<32> went from 263 to 197 us).  L is the transform length along k1.  Both sums over q run over
// -N_k < q < N_k, in terms of |q| since T is even.  A pair costs 4 N_k^4 multiply-adds per
// nucleus, as many as the Toeplitz products of one of its x-points.
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_fft.hpp"
#include "chasm_theta.hpp"

namespace chasm {

// One thread per (row of N_k factors, k).
template <int NK>
__global__ __launch_bounds__(256) void k_theta_mod(fft::cd* __restrict__ et, const ThetaArgs a)
{
    const int nrow = a.nx[0] + a.nx[1] + a.nx[2];
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= (long long)NK * (4 + (long long)a.nnuc * nrow)) return;
    const int k = (int)(t % NK);
    const long long r = t / NK;
    double ph;
    if (r < 4) {
        ph = 3.14159265358979323846 * (double)t / (2 * NK);
    } else {
        const int nu = (int)((r - 4) / nrow);
        int i = (int)((r - 4) % nrow), d = 0;
        while (d < 2 && i >= a.nx[d]) i -= a.nx[d++];
        const double xc = a.x_lo[d] + i * a.hx[d];
        ph = 2.0 * (xc - a.xa[nu][d]) * a.hk[d] * k;
    }
    double s, c;
    sincos(ph, &s, &c);
    et[t] = fft::cd{c, -s};
}

// (2 if q > 0) cos(phi q - 2 pi n q / (4 N_k)) from the node's row e^{-i phi q}.
template <int NK>
__device__ __forceinline__ double shifted_cos(const fft::cd* et, const fft::cd* row, int q, int n)
{
    const fft::cd e = row[q], w = et[(n * q) % (4 * NK)];
    return (q ? 2.0 : 1.0) * fma(e.re, w.re, e.im * w.im);
}

// U of the nodes i1_0 .. : block (i1, nu; 4 frequencies m), a thread per (q2, q3).
template <int NK>
__global__ __launch_bounds__(256) void k_theta_u(double* __restrict__ U, const double* __restrict__ T,
                                                const fft::cd* __restrict__ et, const ThetaArgs a, int i1_0)
{
    constexpr int P = 2 * NK;
    __shared__ double cs[4][NK];
    const int il = blockIdx.x / a.nnuc, nu = blockIdx.x % a.nnuc, m0 = 4 * blockIdx.y;
    const fft::cd* row = mod_row(et, a, NK, nu, 0, i1_0 + il);
    for (int t = threadIdx.x; t < 4 * NK; t += 256)
        cs[t / NK][t % NK] = a.wgt[nu] * shifted_cos<NK>(et, row, t % NK, 2 * (m0 + t / NK) + 1);
    __syncthreads();
    double* out = U + ((long long)blockIdx.x * P + m0) * (NK * NK);
    for (int t = threadIdx.x; t < NK * NK; t += 256) {
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int q = 0; q < NK; ++q) {
            const double x = T[q * (NK * NK) + t];
            for (int m = 0; m < 4; ++m) s[m] = fma(cs[m][q], x, s[m]);
        }
        for (int m = 0; m < 4; ++m) out[m * (NK * NK) + t] = s[m];
    }
}

// Where a table line keeps q3 (even) and q3 + 1 of xi2.
template <int NK>
__device__ __forceinline__ int line_at(int q, int xi2)
{
    return (q / 2 * (2 * NK) + (xi2 & 1) * NK + xi2 / 2) * 2;
}

// D and S of the pairs p0 ..: block (pair, nu; 4 planes c).  A thread sums one q3 of a
// plane at four couples (xi2, P - xi2), (0, N_k) for the first: those are closed under the
// negation of both frequencies, so four sums give D and S of both.  Neighbours in q3 then
// exchange halves, so that each writes q3 pairs.  A 128 MiB range takes 46 us at N_k = 16;
// with four q3 of one couple to a thread, which needs no exchange, 53 (and 103 for 38 at
// N_k = 32, 23 pairs of two nuclei): its loads of U serve fewer sums.
template <int NK>
__global__ __launch_bounds__(256) void k_theta_table(double* __restrict__ tab, const double* __restrict__ U,
                                                    const fft::cd* __restrict__ et, const ThetaArgs a, int p0,
                                                    int i1_0, int L)
{
    constexpr int P = 2 * NK, RS = NK + 1, G = 4;
    __shared__ double c2[P * RS];                        // [xi2][q2]
    const int pair = p0 + blockIdx.x / a.nnuc, nu = blockIdx.x % a.nnuc;
    const int i1 = pair / a.nx[1], i2 = pair % a.nx[1];
    const fft::cd* row = mod_row(et, a, NK, nu, 1, i2);
    for (int t = threadIdx.x; t < P * NK; t += 256)
        c2[t / NK * RS + t % NK] = shifted_cos<NK>(et, row, t % NK, 2 * (t / NK));
    __syncthreads();
    const double* Ui = U + ((long long)(i1 - i1_0) * a.nnuc + nu) * P * (NK * NK);
    for (int task = threadIdx.x; task < NK * NK; task += 256) {
        const int q = task % NK, g0 = task / NK % (NK / G) * G, c = 4 * blockIdx.y + task / (NK * (NK / G));
        const int m = c / L + P / L * (c % L);
        const double* up = Ui + m * (NK * NK) + q;
        const double* um = Ui + (P - 1 - m) * (NK * NK) + q;
        double px[G] = {}, py[G] = {}, mx[G] = {}, my[G] = {};
#pragma unroll 4
        for (int b = 0; b < NK; ++b) {
            const double u = up[b * NK], v = um[b * NK];
            for (int g = 0; g < G; ++g) {
                const int x = g0 + g;
                const double cx = c2[x * RS + b], cy = c2[(x ? P - x : NK) * RS + b];
                px[g] = fma(u, cx, px[g]);
                py[g] = fma(u, cy, py[g]);
                mx[g] = fma(v, cx, mx[g]);
                my[g] = fma(v, cy, my[g]);
            }
        }
        double* out = tab + ((long long)blockIdx.x * NK + c) * P * P;
        const bool odd = q & 1;                          // even lanes write xi2 = x, odd ones xi2 = y
        for (int g = 0; g < G; ++g) {
            const int x = g0 + g, y = x ? P - x : NK;
            const double nx = x ? my[g] : mx[g], ny = x ? mx[g] : my[g];   // at the negated frequencies
            const double xd = px[g] - nx, xs = px[g] + nx, yd = py[g] - ny, ys = py[g] + ny;
            const double d = __shfl_xor(odd ? xd : yd, 1), s = __shfl_xor(odd ? xs : ys, 1);
            double2* o = reinterpret_cast<double2*>(out + line_at<NK>(q & ~1, odd ? y : x));
            o[0] = odd ? make_double2(d, yd) : make_double2(xd, d);
            o[NK * P / 2] = odd ? make_double2(s, ys) : make_double2(xs, s);
        }
    }
}

}  // namespace chasm
