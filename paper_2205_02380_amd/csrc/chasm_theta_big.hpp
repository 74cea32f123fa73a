// chasm_theta_big.hpp -- the truncated-kernel evaluation of Theta_V (Sec. 4, eq. 4.6
// with the tensor of eq. 4.9) for k-grids whose per-x-point intermediate does not fit
// in one CU (N_k = 32 and 64; also built for 16 to check it against the one-block form
// of chasm_theta_plane.hpp).  Same mathematics as k_theta:
//   Theta(x, k_p) = sum_a w_a Im( e^{i phi_a.p} [circular convolution of period
//                   P = 2 N_k of T with the zero-padded e^{-i phi_a.p'} f_p'](p) ),
// evaluated in three stages over a batch of x-points, with a complex FP64
// intermediate in device memory, W[x][xi1][k3][k2]:
//   k_thA    modulate each k1 line and transform it along k1 (zero padded to P);
//   k_thBCD  per (x, xi1): transform along k2 (zero padded), the Toeplitz product
//            along k3 with K(xi1, xi2, |q3|) (the kernel transformed along k1 and k2,
//            see tensor_partial), and the inverse along k2 (first N_k outputs);
//   k_thE    inverse along k1 (first N_k outputs), demodulate, take the imaginary
//            part, accumulate over the nuclei.
// Every P-point transform of a zero-padded line, and every inverse restricted to the
// first N_k outputs, is split by residue: output (input) index S f + h, f < 32,
// h < S = P / 32, is a 32-point transform of the twiddled line folded modulo 32, so
// each work item of A and E holds 32 complex values in registers.  The field is in x-major
// order [b][x][k3][k2][k1], as for k_theta.  The modulations are per-axis factors of the
// handle's table: k1 and k3 in A and E, k2 in k_thBCD.
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_fft.hpp"
#include "chasm_theta.hpp"
#include "chasm_theta_plane.hpp"

namespace chasm {

template <int NK>
struct BigShape {
    static constexpr int P = 2 * NK;
    static constexpr int L = 32;              // transform length of a work item
    static constexpr int S = P / L;           // residues
    static constexpr int RS = NK + 1;         // padded LDS row (complex)
    static constexpr int LA = 256;            // k1 lines (threads) per block in A
    static constexpr int LE = NK <= 32 ? 256 : 64;          // and in E
    static constexpr int NTB = 2 * NK > 64 ? 2 * NK : 64;   // threads of k_thBCD
    static_assert(P % L == 0 && NK * NK % LA == 0 && LE % NK == 0, "shape");
};

// The factors that A and E apply along k1 on this thread's line (row k3): entry j =
// e^{-i phi_1 j} e^{-i phi_3 k3} (the k2 factor rides on the twiddles of B and D), for
// residue h = 0, times wgt; next_residue multiplies by w^j.
template <int NK>
__device__ __forceinline__ LineFactors<NK> big_factors(const ModRows& e, int k3, double wgt = 1.0)
{
    LineFactors<NK> f;
    const fft::cd e3 = {wgt * e.e3[k3].re, wgt * e.e3[k3].im};
    fft::sfor<0, NK / 16>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        f.v[q] = fft::cmul(e.e1[threadIdx.x % 16 + 16 * q], e3);
    });
    return f;
}

template <int NK>
__device__ __forceinline__ void next_residue(LineFactors<NK>& f, const fft::cd* et)
{
    fft::sfor<0, NK / 16>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        f.v[q] = fft::cmul(f.v[q], et[threadIdx.x % 16 + 16 * q]);
    });
}

// ---- A: k1 forward.  Block = 256 k1 lines of one x-point, a thread per line and one
// residue h (outputs xi1 = S f + h) at a time: 32 complex values in registers.
template <typename T, int NK>
__global__ __launch_bounds__(BigShape<NK>::LA, 2) void k_thA(const T* __restrict__ fx, fft::cd* __restrict__ W,
                                                            const fft::cd* __restrict__ et, const ThetaArgs a,
                                                            long long x0, int nu)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, S = B::S, BPX = NK * NK / B::LA;
    const long long xl = blockIdx.x / BPX;
    const int l0 = (int)(blockIdx.x % BPX) * B::LA, la = l0 + threadIdx.x;   // k3 * NK + k2
    LineFactors<NK> lf = big_factors<NK>(mod_rows_at<NK>(et, a, x0 + xl, nu), la / NK);
    const T* line = fx + (x0 + xl) * (long long)(NK * NK * NK) + (long long)la * NK;
    cd* out = W + xl * (long long)(P * NK * NK) + la;
#pragma unroll 1
    for (int h = 0; h < S; ++h) {
        cd y[32];
        // y[k mod 32] = sum e^{-i phi.p} f(p) w^{h k}, k = k1 < NK (zero padded to P)
        sfor<0, (NK + 31) / 32>([&](auto sc) {
            constexpr int k0 = decltype(sc)::value * 32, n = NK < 32 ? NK : 32;
            double fv[n];
            load_k1<T, n>(line + k0, fv);
            sfor<0, n>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                const cd m = lf.template at<k0 + k>();
                if constexpr (k0 == 0) y[k] = cd{m.re * fv[k], m.im * fv[k]};
                else y[k] = cd{fma(m.re, fv[k], y[k].re), fma(m.im, fv[k], y[k].im)};
            });
        });
        if constexpr (NK < 32) sfor<NK, 32>([&](auto kc) { y[decltype(kc)::value] = cd{0.0, 0.0}; });
        transform<32, -1>(y);
        sfor<0, 32>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            out[(long long)(S * f + h) * (NK * NK)] = y[f];   // xi1 = S f + h
        });
        next_residue<NK>(lf, et);
    }
}

// ---- B, C, D for N_k <= 32: planes W[x][xi1][k3][k2] through plane_conv, in place; a
// one-wave block takes 64 / (2 N_k) planes, and no lane waits for another wave.  At
// N_k = 32 a lane's half line (32 complex values) and the Toeplitz sums fill 256 VGPRs: two
// waves per SIMD, FP64 VALU bound.  Per 2048 x-points: 1.38 ms, against 2.26 ms for one
// wave per SIMD with half the lanes idle in B and D; k_thA 0.43 (0.61), k_thE 0.58 (0.87).
template <int NK>
__global__ __launch_bounds__(64, 2) void k_thBCD_plane(fft::cd* __restrict__ W, const double* __restrict__ kt,
                                                      const fft::cd* __restrict__ et, const ThetaArgs a,
                                                      long long x0, int nu)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    constexpr int P = S::P, RS = S::RS, PPB = 64 / S::LANES;
    __shared__ cd slots[PPB * S::SLOT];
    const int lane = threadIdx.x % S::LANES, k3 = lane % NK, h = lane / NK, grp = threadIdx.x / S::LANES;
    const long long p = (long long)blockIdx.x * PPB + grp;
    const int xi1 = (int)(p % P);
    cd* plane = W + p * (long long)(NK * NK);
    cd* slot = slots + grp * S::SLOT;
    // a block's planes belong to one x-point (PPB divides P)
    LineFactors<NK> tw = half_factors<NK>(et, mod_rows_at<NK>(et, a, x0 + p / P, nu).e2, h, lane, nullptr);
    sfor<0, NK / 2>([&](auto ic) {   // two rows per step
        constexpr int i = decltype(ic)::value;
        slot[(2 * i + h) * RS + k3] = plane[2 * i * NK + lane];
    });
    __syncthreads();
    plane_conv<NK>(slot, kt + ((long long)xi1 * P + 2 * k3 + h) * NK, tw, k3, h);
    __syncthreads();
    sfor<0, NK / 2>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        plane[2 * i * NK + lane] = slot[(2 * i + h) * RS + k3];
    });
}

// ---- B, C, D for N_k = 64: one block per (x-point, xi1) slice W[x][xi1][k3][k2] (in place).
template <int NK>
__global__ __launch_bounds__(BigShape<NK>::NTB) void k_thBCD(fft::cd* __restrict__ W, const double* __restrict__ kt,
                                                              const fft::cd* __restrict__ et, const ThetaArgs a,
                                                              long long x0, int nu)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, L = B::L, S = B::S, RS = B::RS, NT = B::NTB;
    constexpr int JC = NK / 16;                 // 16-output chunks of a Toeplitz row
    __shared__ cd ACC[NK * RS];                 // [j3][j2]: k2 inverse, summed over residues
    __shared__ cd BC[L * RS];                   // [f][k3]: k2 forward of residue h
    __shared__ cd OC[L * RS];                   // [f][j3]: after the k3 Toeplitz product
    __shared__ double KK[L * RS];               // [f][q3]: K(xi1, S f + h, q3)
    __shared__ cd TW[S][NK];                    // e^{-i phi_2 k} w^{h k}
    const long long xl = blockIdx.x / P;
    const int xi1 = (int)(blockIdx.x % P);
    cd* slice = W + (xl * P + xi1) * (long long)(NK * NK);
    const int tid = threadIdx.x;
    const cd* e2 = mod_rows_at<NK>(et, a, x0 + xl, nu).e2;
    for (int t = tid; t < S * NK; t += NT) TW[t / NK][t % NK] = cmul(e2[t % NK], et[((t / NK) * (t % NK)) % P]);
    __syncthreads();

    sfor<0, S>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        // B: the k2 forward transform of every k3 row, outputs xi2 = S f + h
        for (int r = tid; r < NK; r += NT) {
            cd y[32];
            sfor<0, 32>([&](auto jc) { y[decltype(jc)::value] = cd{0.0, 0.0}; });
            const cd* row = slice + (long long)r * NK;
            sfor<0, NK>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                y[k % 32] = cadd(y[k % 32], cmul(row[k], TW[h][k]));
            });
            transform<32, -1>(y);
            sfor<0, 32>([&](auto fc) { BC[decltype(fc)::value * RS + r] = y[decltype(fc)::value]; });
        }
        for (int t = tid; t < L * NK; t += NT) {
            const int f = t / NK, q = t % NK;
            KK[f * RS + q] = kt[((long long)xi1 * P + (S * f + h)) * NK + q];
        }
        __syncthreads();
        // C: o_j = sum_i K(|j - i|) row_i for each row f, 16 outputs per work item;
        // the 16 kernel values of one input form a window that slides down by one
        for (int t = tid; t < L * JC; t += NT) {
            const int f = t % L, j0 = (t / L) * 16;
            const double* kk = KK + f * RS;
            const cd* row = BC + f * RS;
            cd o[16];
            double w[16];
            sfor<0, 16>([&](auto jc) {
                constexpr int jj = decltype(jc)::value;
                o[jj] = cd{0.0, 0.0};
                w[jj] = kk[j0 + jj];            // window of input i = 0: K(|j0 + jj - 0|)
            });
            sfor<0, NK>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const cd r = row[i];
                sfor<0, 16>([&](auto jc) {
                    constexpr int jj = decltype(jc)::value;
                    o[jj].re = fma(w[jj], r.re, o[jj].re);
                    o[jj].im = fma(w[jj], r.im, o[jj].im);
                });
                if constexpr (i + 1 < NK) {
                    // window of input i + 1: K(|j0 + jj - i - 1|) = previous window shifted
                    sfor<0, 15>([&](auto jc) {
                        constexpr int jj = 15 - decltype(jc)::value;
                        w[jj] = w[jj - 1];
                    });
                    const int m = j0 - i - 1;
                    w[0] = kk[m < 0 ? -m : m];
                }
            });
            sfor<0, 16>([&](auto jc) { OC[f * RS + j0 + decltype(jc)::value] = o[decltype(jc)::value]; });
        }
        __syncthreads();
        // D: inverse along k2 over this residue's xi2, first NK outputs, summed over the
        // residues
        for (int j3 = tid; j3 < NK; j3 += NT) {
            cd v[32];
            sfor<0, 32>([&](auto fc) { v[decltype(fc)::value] = OC[decltype(fc)::value * RS + j3]; });
            transform<32, +1>(v);
            sfor<0, NK>([&](auto jc) {
                constexpr int j2 = decltype(jc)::value;
                const cd x = cmul(v[j2 % 32], conj(TW[h][j2]));
                ACC[j3 * RS + j2] = h == 0 ? x : cadd(ACC[j3 * RS + j2], x);
            });
        }
        __syncthreads();
    });
    for (int t = tid; t < NK * NK; t += NT) {
        const int j3 = t / NK, j2 = t % NK;
        slice[t] = ACC[j3 * RS + j2];
    }
}

// ---- E: k1 inverse, demodulation, imaginary part, sum over nuclei (the weight is
// already in).  A thread per k1 line, one residue at a time; the real result of a line
// is kept in registers (LDS at N_k = 64).  first: no earlier nucleus; last: write the
// result (type T) to fx, else keep the FP64 sum in acc.
template <typename T, int NK>
__global__ __launch_bounds__(BigShape<NK>::LE, 2) void k_thE(const fft::cd* __restrict__ W, double* __restrict__ acc,
                                                            T* __restrict__ fx, const fft::cd* __restrict__ et,
                                                            const ThetaArgs a, long long x0, int nu, int first, int last)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, S = B::S, RS = B::RS, BPX = NK * NK / B::LE;
    constexpr bool REG = NK <= 32;
    __shared__ double TH[REG ? 1 : B::LE * RS];
    const long long xl = blockIdx.x / BPX;
    const int l0 = (int)(blockIdx.x % BPX) * B::LE, la = l0 + threadIdx.x;   // j3 * NK + j2
    LineFactors<NK> lf = big_factors<NK>(mod_rows_at<NK>(et, a, x0 + xl, nu), la / NK, a.wgt[nu]);
    const cd* src = W + xl * (long long)(P * NK * NK) + la;
    const long long off = (x0 + xl) * (long long)(NK * NK * NK) + (long long)la * NK;
    double* ac = acc + xl * (long long)(NK * NK * NK) + (long long)la * NK;
    double thr[REG ? NK : 1];
    double* th = TH + (REG ? 0 : threadIdx.x * RS);
    auto at = [&](auto jc) -> double& {
        if constexpr (REG) return thr[decltype(jc)::value];
        else return th[decltype(jc)::value];
    };
    sfor<0, NK>([&](auto jc) { at(jc) = first ? 0.0 : ac[decltype(jc)::value]; });
#pragma unroll 1
    for (int h = 0; h < S; ++h) {
        cd v[32];
        sfor<0, 32>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            v[f] = src[(long long)(S * f + h) * (NK * NK)];
        });
        transform<32, +1>(v);
        sfor<0, NK>([&](auto jc) {
            constexpr int j1 = decltype(jc)::value;
            const cd m = lf.template at<j1>();
            at(jc) = fma(m.re, v[j1 % 32].im, fma(-m.im, v[j1 % 32].re, at(jc)));   // Im(conj(m) v)
        });
        next_residue<NK>(lf, et);
    }
    if (last) {
        sfor<0, (NK + 31) / 32>([&](auto sc) {
            constexpr int k0 = decltype(sc)::value * 32, n = NK < 32 ? NK : 32;
            double o[n];
            sfor<0, n>([&](auto jc) { o[decltype(jc)::value] = at(std::integral_constant<int, k0 + decltype(jc)::value>{}); });
            store_k1<T, n>(fx + off + k0, o);
        });
    } else {
        sfor<0, NK>([&](auto jc) { ac[decltype(jc)::value] = at(jc); });
    }
}

}  // namespace chasm
