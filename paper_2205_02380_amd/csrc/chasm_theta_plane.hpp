// chasm_theta_plane.hpp -- the (k2, k3) part of the truncated-kernel convolution of
// Theta_V on one (x, xi1) plane by 2 N_k lanes of one wave, and the one-block kernel
// built on it (N_k = 8 and 16).  Mathematics and notation as in chasm_theta.hpp.
//
// A plane is N_k rows (k3) of N_k complex values (k2).  Its work is
//   B  per row: k2 forward transform, zero-padded to P = 2 N_k outputs xi2 = 2 f + h:
//      the N_k-point transform of row_j w^{h j}, h = 0, 1;
//   C  per xi2: the N_k x N_k real symmetric Toeplitz product along k3;
//   D  per row: k2 inverse, first N_k outputs: the sum over h of the N_k-point inverse of
//      the xi2 = 2 f + h inputs times w^{-h j}.
// Lane (h, k3) does B and D of row k3 for its h, and C of line xi2 = 2 k3 + h, so all
// 2 N_k lanes are busy in every stage with one N_k-point line each (2 N_k VGPR pairs).
// Only lanes of one wave share a plane, so nothing but the two transposes between rows
// and lines orders them: those go through the plane's own LDS slot, real parts and then
// imaginary parts (K is real, so the two parts of C are independent), 2 N_k lines of
// N_k doubles -- exactly the slot's size.  The sum over h exchanges half of each line
// with the partner lane, after which each lane holds N_k/2 outputs of its row.
// Twiddles that a lane needs for its own h come from LDS with the modulation along k2
// folded in.
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_fft.hpp"
#include "chasm_theta.hpp"

namespace chasm {

template <int NK>
struct PlaneShape {
    static constexpr int P = 2 * NK;
    static constexpr int RS = NK + 1;        // padded row: NK + 1 complex, or NK + 1 doubles per line
    static constexpr int SLOT = NK * RS;     // complex values per plane
    static constexpr int LANES = 2 * NK;     // lanes per plane
    static_assert(LANES <= 64, "a plane belongs to one wave");
};

// Orders this wave's LDS accesses as written (they execute in order; this keeps the
// compiler from reordering accesses whose cross-lane dependence it cannot see).
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// x + x' of the lanes l and l ^ NK: the lane with h = 0 (bit NK of the lane index clear)
// gets the sum of the partners' `a`, the lane with h = 1 the sum of their `b`.
template <int NK>
__device__ __forceinline__ double pair_sum(double a, double b, int h)
{
    if constexpr (NK == 8) {
        const double keep = h ? b : a, send = h ? a : b;
        const int lo = __builtin_amdgcn_mov_dpp(__double2loint(send), 0x128, 0xF, 0xF, false);   // row_ror:8
        const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(send), 0x128, 0xF, 0xF, false);
        return keep + __hiloint2double(hi, lo);
    } else {
        const unsigned alo = (unsigned)__double2loint(a), ahi = (unsigned)__double2hiint(a);
        const unsigned blo = (unsigned)__double2loint(b), bhi = (unsigned)__double2hiint(b);
        if constexpr (NK == 16) {   // odd 16-lane rows of a <-> even rows of b
            const auto lo = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
            return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
        } else {                    // upper 32 lanes of a <-> lower 32 of b
            static_assert(NK == 32, "lane exchange");
            const auto lo = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
            return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
        }
    }
}

// o = K x for the symmetric Toeplitz matrix K[j][i] = kk[|j - i|], sixteen outputs at a
// time (bounds the accumulators at N_k = 32).
template <int NK>
__device__ __forceinline__ void toeplitz_line(const double (&kk)[NK], double* line)
{
    constexpr int JB = NK < 16 ? NK : 16;
    double x[NK];
    fft::sfor<0, NK>([&](auto ic) { x[decltype(ic)::value] = line[decltype(ic)::value]; });
    fft::sfor<0, NK / JB>([&](auto bc) {
        constexpr int j0 = decltype(bc)::value * JB;
        double o[JB];
        fft::sfor<0, JB>([&](auto jc) { o[decltype(jc)::value] = 0.0; });
        fft::sfor<0, NK>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            fft::sfor<0, JB>([&](auto jc) {
                constexpr int j = j0 + decltype(jc)::value;
                constexpr int d = j > i ? j - i : i - j;
                o[j - j0] = fma(kk[d], x[i], o[j - j0]);
            });
        });
        fft::sfor<0, JB>([&](auto jc) { line[j0 + decltype(jc)::value] = o[decltype(jc)::value]; });
    });
}

// Stages B, C, D of the plane in `slot`, in place.  k3, h: this lane's row and half;
// kt: the kernel values K(xi1, 2 k3 + h, 0 .. N_k - 1) of this lane's line; twf, twd: the
// factors of this lane's half, row_j -> row_j twf_j before B and out_j -> out_j twd_j
// after D.
template <int NK>
__device__ __forceinline__ void plane_conv(fft::cd* slot, const double* __restrict__ kt, const fft::cd* twf,
                                           const fft::cd* twd, int k3, int h)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    double kk[NK];
    const double2* kr = reinterpret_cast<const double2*>(kt);
    sfor<0, NK / 2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const double2 t = kr[q];
        kk[2 * q] = t.x;
        kk[2 * q + 1] = t.y;
    });
    cd y[NK];
    cd* row = slot + k3 * S::RS;
    sfor<0, NK>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        y[j] = cmul(row[j], twf[j]);
    });
    transform<NK, -1>(y);
    wave_order();
    double* col = reinterpret_cast<double*>(slot) + h * NK * S::RS + k3;      // row k3 of half h: stride RS
    double* line = reinterpret_cast<double*>(slot) + (h * NK + k3) * S::RS;   // line xi2 = 2 k3 + h
    sfor<0, NK>([&](auto fc) { col[decltype(fc)::value * S::RS] = y[decltype(fc)::value].re; });
    wave_order();
    toeplitz_line<NK>(kk, line);
    wave_order();
    sfor<0, NK>([&](auto fc) { y[decltype(fc)::value].re = col[decltype(fc)::value * S::RS]; });
    wave_order();
    sfor<0, NK>([&](auto fc) { col[decltype(fc)::value * S::RS] = y[decltype(fc)::value].im; });
    wave_order();
    toeplitz_line<NK>(kk, line);
    wave_order();
    sfor<0, NK>([&](auto fc) { y[decltype(fc)::value].im = col[decltype(fc)::value * S::RS]; });
    wave_order();
    transform<NK, +1>(y);
    sfor<0, NK>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        y[j] = cmul(y[j], twd[j]);
    });
    constexpr int H = NK / 2;
    sfor<0, H>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        row[h * H + j] = cd{pair_sum<NK>(y[j].re, y[j + H].re, h), pair_sum<NK>(y[j].im, y[j + H].im, h)};
    });
}

// Modulation table of a handle: the P factors w^j = e^{-2 pi i j / P}, then for every
// nucleus the rows e^{-i phi k} (k < N_k, phi = 2 (x - x_a) hk) of the nx1 + nx2 + nx3
// nodes of the three axes.  One thread per (row of N_k factors, k).
template <int NK>
__global__ __launch_bounds__(256) void k_theta_mod(fft::cd* __restrict__ et, const ThetaArgs a)
{
    const int nrow = a.nx[0] + a.nx[1] + a.nx[2];
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    if (t >= (long long)NK * (2 + (long long)a.nnuc * nrow)) return;
    const int k = (int)(t % NK);
    const long long r = t / NK;
    double ph;
    if (r < 2) {
        ph = 3.14159265358979323846 * (double)t / NK;
    } else {
        const int nu = (int)((r - 2) / nrow);
        int i = (int)((r - 2) % nrow), d = 0;
        while (d < 2 && i >= a.nx[d]) i -= a.nx[d++];
        const double xc = a.x_lo[d] + i * a.hx[d];
        ph = 2.0 * (xc - a.xa[nu][d]) * a.hk[d] * k;
    }
    double s, c;
    sincos(ph, &s, &c);
    et[t] = fft::cd{c, -s};
}

// The rows of the modulation table at x-point xp (batch members stacked) for nucleus nu.
struct ModRows {
    const fft::cd *e1, *e2, *e3;
};

template <int NK>
__device__ __forceinline__ ModRows mod_rows_at(const fft::cd* et, const ThetaArgs& a, long long xp, int nu)
{
    const unsigned loc = (unsigned)(xp % (unsigned)a.npts);
    const unsigned i1 = loc % (unsigned)a.nx[0], up = loc / (unsigned)a.nx[0];
    const unsigned i2 = up % (unsigned)a.nx[1], i3 = up / (unsigned)a.nx[1];
    const fft::cd* e = et + 2 * NK + (long long)nu * (a.nx[0] + a.nx[1] + a.nx[2]) * NK;
    return {e + i1 * NK, e + (a.nx[0] + i2) * NK, e + (a.nx[0] + a.nx[1] + i3) * NK};
}

// One x-point per block at a time (persistent over x-points), N_k^2 threads, FP64
// throughout.  The xi1 axis goes by parity: chunk r holds xi1 = r + 2 m (m < N_k), the
// N_k-point transform of line_j e^{-i phi_1 j} w^{r j}.  Per chunk:
//   A  thread (k2, k3): modulated k1 line, N_k-point transform      -> plane m, [k3][k2]
//   BCD  plane_conv on the N_k planes, 2 N_k lanes each
//   E  thread (k2, k3): N_k-point inverse over the planes, demodulated, into the real
//      result the thread keeps in registers (16 doubles at N_k = 16)
// The modulations are products of per-axis factors: e02 = e^{-i phi_1 j} w^{r j}
// e^{-i phi_3 k3} is formed once per x-point and chunk (one entry per thread) and used by
// A and, conjugated, by E; the k2 factor rides on the twiddles of B and D (and D's
// carry the nucleus weight).
//
// Bound: FP64 VALU (about 1.2e6 lane instructions per x-point at N_k = 16, 44 % of them
// the Toeplitz products: 7 ms on 61^3 x-points at full rate) against 1.6 MB of LDS
// traffic per x-point.  The planes of a chunk take 70 KB at N_k = 16, so two blocks (two
// waves per SIMD, 196 VGPRs each) share a CU and one's barriers and LDS waits hide
// behind the other.  Measured on 61^3 x 16^3, FP32 field: 14.7 ms, against 22.1 ms for a
// form with the chunk's k2-transformed planes side by side in LDS (140 KB, one wave per
// SIMD, a barrier after every stage).
template <typename T, int NK>
__global__ __launch_bounds__(NK * NK, 2) void k_theta(T* __restrict__ fx, const double* __restrict__ kt,
                                                     const fft::cd* __restrict__ et, const ThetaArgs a,
                                                     long long total)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    constexpr int NT = NK * NK, P = S::P, RS = S::RS;
    constexpr int GROUPS = NT / S::LANES;            // planes worked on at a time
    __shared__ cd W[NK * S::SLOT];
    __shared__ cd E02[2][NK * NK];                   // [r][k3][j]
    __shared__ cd TWF[2][NK], TWD[2][NK];            // [h][k2]

    const int tid = threadIdx.x;
    const int c2 = tid % NK, c3 = tid / NK;          // k1 line (k2, k3) of stages A and E
    const int k3 = tid % NK, h = (tid / NK) & 1, grp = tid / S::LANES;

    for (long long xp = blockIdx.x; xp < total; xp += gridDim.x) {
        T* line = fx + xp * (long long)(NK * NK * NK) + tid * NK;
        double th[NK];
        sfor<0, NK>([&](auto jc) { th[decltype(jc)::value] = 0.0; });

        for (int nu = 0; nu < a.nnuc; ++nu) {
            const ModRows e = mod_rows_at<NK>(et, a, xp, nu);
            __syncthreads();   // the previous pass no longer reads the factors
            {
                const cd b = cmul(e.e1[c2], e.e3[c3]);   // j = c2 here
                E02[0][tid] = b;
                E02[1][tid] = cmul(b, et[c2]);
            }
            if (tid < 2 * NK) {
                const int hh = tid / NK, j = tid % NK;
                const cd f = hh ? cmul(e.e2[j], et[j]) : e.e2[j];
                TWF[hh][j] = f;
                TWD[hh][j] = cd{a.wgt[nu] * f.re, -a.wgt[nu] * f.im};
            }
            __syncthreads();
#pragma unroll 1
            for (int r = 0; r < 2; ++r) {
                {   // A
                    double fv[NK];
                    load_k1<T, NK>(line, fv);
                    cd y[NK];
                    sfor<0, NK>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const cd m = E02[r][c3 * NK + j];
                        y[j] = cd{m.re * fv[j], m.im * fv[j]};
                    });
                    transform<NK, -1>(y);
                    sfor<0, NK>([&](auto mc) {
                        constexpr int m = decltype(mc)::value;
                        W[m * S::SLOT + c3 * RS + c2] = y[m];
                    });
                }
                __syncthreads();
#pragma unroll 1
                for (int m = grp; m < NK; m += GROUPS)   // B, C, D: xi1 = r + 2 m, xi2 = 2 k3 + h
                    plane_conv<NK>(W + m * S::SLOT, kt + ((long long)(r + 2 * m) * P + 2 * k3 + h) * NK, TWF[h],
                                   TWD[h], k3, h);
                __syncthreads();
                {   // E
                    cd y[NK];
                    sfor<0, NK>([&](auto mc) {
                        constexpr int m = decltype(mc)::value;
                        y[m] = W[m * S::SLOT + c3 * RS + c2];
                    });
                    transform<NK, +1>(y);
                    sfor<0, NK>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const cd m = E02[r][c3 * NK + j];
                        th[j] = fma(m.re, y[j].im, fma(-m.im, y[j].re, th[j]));   // Im(conj(m) y)
                    });
                }
            }
        }
        store_k1<T, NK>(line, th);
    }
}

}  // namespace chasm
