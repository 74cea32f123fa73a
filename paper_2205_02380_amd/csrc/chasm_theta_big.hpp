// chasm_theta_big.hpp -- the convolution of Theta_V for k-grids whose per-x-point
// intermediate does not fit in one CU (N_k = 32 and 64; also built for 16 to check it
// against the one-block form of chasm_theta_plane.hpp).  Mathematics, notation and the
// order of the x-points as in chasm_theta.hpp; three stages over a batch of x-points, with
// a complex FP64 intermediate in device memory, W[x][c][k3][k2], c < N_k the held planes:
//   k_thA    transform each k1 line along k1 (zero padded to P);
//   k_thBCD  per (x, c): transform along k2 (zero padded), the even and the odd Toeplitz
//            matrix along k3, and the inverse along k2 (first N_k outputs);
//   k_thE    inverse along k1 (first N_k outputs), real part.
// The k1 frequencies are split by residue: m = S f + h, f < L, h < S = P / L, is an
// L-point transform of the line times e^{-2 pi i (h + 1/2) j / P}, folded modulo L.  The
// conjugate of residue h is S - 1 - h, so the residues h < S / 2 are held, plane c = L h + f,
// and each work item of A and E has L complex values in registers.  The k2 transforms of
// k_thBCD are split likewise.
#pragma once
#include <hip/hip_runtime.h>

#include "chasm_fft.hpp"
#include "chasm_theta.hpp"
#include "chasm_theta_plane.hpp"
#include "chasm_theta_table.hpp"

namespace chasm {

template <int NK>
struct BigShape {
    static constexpr int P = 2 * NK;
    static constexpr int L = NK < 32 ? NK : 32;             // transform length of a work item
    static constexpr int S = P / L;                         // residues
    static constexpr int RS = NK + 1;                       // padded LDS row (complex)
    static constexpr int LA = 256;                          // k1 lines (threads) per block in A
    static constexpr int LE = NK <= 32 ? 256 : 64;          // and in E
    static constexpr int NTB = 2 * NK > 64 ? 2 * NK : 64;   // threads of k_thBCD
    static_assert(P % L == 0 && S % 2 == 0 && NK * NK % LA == 0 && LE % NK == 0, "shape");
};

// ---- A: k1 forward.  Block = 256 k1 lines of one x-point, a thread per line.
template <typename T, int NK>
__global__ __launch_bounds__(BigShape<NK>::LA, 2) void k_thA(const T* __restrict__ fx, fft::cd* __restrict__ W,
                                                            const ThetaArgs a, unsigned t0)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, S = B::S, L = B::L, BPX = NK * NK / B::LA;
    const unsigned xl = blockIdx.x / BPX;
    const int la = (int)(blockIdx.x % BPX) * B::LA + threadIdx.x;            // k3 * NK + k2
    const T* line = fx + x_point(a, t0 + xl).xp * (NK * NK * NK) + (long long)la * NK;
    cd* out = W + xl * (long long)(NK * NK * NK) + la;
    sfor<0, S / 2>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        cd y[L];
        asm volatile("" ::: "memory");       // the line is read again, not kept (128 registers at N_k = 64)
        sfor<0, NK / L>([&](auto sc) {
            constexpr int k0 = decltype(sc)::value * L;
            double fv[L];
            load_k1<T, L>(line + k0, fv);
            sfor<0, L>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                constexpr cd m = twiddle((2 * h + 1) * (k0 + k), 2 * P, -1);
                if constexpr (k0 == 0) y[k] = cd{m.re * fv[k], m.im * fv[k]};
                else y[k] = cd{fma(m.re, fv[k], y[k].re), fma(m.im, fv[k], y[k].im)};
            });
        });
        transform<L, -1>(y);
        sfor<0, L>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            out[(long long)(L * h + f) * (NK * NK)] = y[f];
        });
    });
}

// ---- B, C, D for N_k <= 32: planes W[x][c][k3][k2] through plane_conv, in place; a
// one-wave block takes 64 / (2 N_k) planes, and no lane waits for another wave.  At
// N_k = 32 a lane's line, its kernel values and the Toeplitz sums are 384 of its 416
// registers: one wave per SIMD.  384 x-points with two nuclei take 194 us (56 % VALU busy), where full
// complex spectra of the modulated field took 490; a loop over planes that requests the next one
// ahead gained 1.5 % of the whole and was left out.
template <int NK>
__global__ __launch_bounds__(64, NK == 32 ? 1 : 2) void k_thBCD_plane(fft::cd* __restrict__ W, const double* __restrict__ tab,
                                                                     const fft::cd* __restrict__ et, const ThetaArgs a,
                                                                     unsigned t0, unsigned p0)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    constexpr int P = S::P, RS = S::RS, PPB = 64 / S::LANES;
    static_assert(NK % PPB == 0, "a block's planes belong to one x-point");
    __shared__ cd slots[PPB * S::SLOT];
    const int lane = threadIdx.x % S::LANES, k3 = lane % NK, h = lane / NK, grp = threadIdx.x / S::LANES;
    const unsigned xl = blockIdx.x / (NK / PPB);
    const int c = (int)(blockIdx.x % (NK / PPB)) * PPB + grp;
    cd* plane = W + ((long long)xl * NK + c) * (NK * NK) + lane;
    cd* slot = slots + grp * S::SLOT;
    const XPoint x = x_point(a, t0 + xl);
    KernelLine kl;
    kl.nnuc = a.nnuc;
    kl.tab = tab + (((long long)(x.pair - p0) * a.nnuc * NK + c) * P) * P + 2 * lane;
    kl.tab_nu = (long long)NK * P * P;
    kl.e3 = mod_row(et, a, NK, 0, 2, x.i3);
    kl.e3_nu = (long long)(a.nx[0] + a.nx[1] + a.nx[2]) * NK;
    LineFactors<NK> tw = half_factors<NK>(et, h, lane, nullptr);
    sfor<0, NK / 2>([&](auto ic) {   // two rows per step
        constexpr int i = decltype(ic)::value;
        slot[(2 * i + h) * RS + k3] = plane[2 * i * NK];
    });
    wave_order();
    plane_conv<NK>(slot, kl, tw, k3, h);
    wave_order();
    sfor<0, NK / 2>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        plane[2 * i * NK] = slot[(2 * i + h) * RS + k3];
    });
}

// ---- B, C, D for N_k = 64: one block per (x-point, c) slice W[x][c][k3][k2] (in place).
template <int NK>
__global__ __launch_bounds__(BigShape<NK>::NTB) void k_thBCD(fft::cd* __restrict__ W, const double* __restrict__ tab,
                                                              const fft::cd* __restrict__ et, const ThetaArgs a,
                                                              unsigned t0, unsigned p0)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, L = B::L, S = B::S, RS = B::RS, NT = B::NTB;
    constexpr int JC = NK / 16;                 // 16-output chunks of a Toeplitz row
    static_assert(L * JC == NT, "one Toeplitz chunk per thread");
    __shared__ cd ACC[NK * RS];                 // [j3][j2]: k2 inverse, summed over residues
    __shared__ cd BC[L * RS];                   // [f][k3]: k2 forward of residue h, then the product
    __shared__ double KD[L * RS], KS[L * RS];   // [f][q3]: even and odd kernel of xi2 = S f + h
    __shared__ cd TW[S][NK];                    // w^{h k}
    const unsigned xl = blockIdx.x / NK;
    const int c = (int)(blockIdx.x % NK);
    cd* slice = W + ((long long)xl * NK + c) * (NK * NK);
    const int tid = threadIdx.x;
    const XPoint x = x_point(a, t0 + xl);
    const double* lines = tab + ((long long)(x.pair - p0) * a.nnuc * NK + c) * P * P;
    for (int t = tid; t < S * NK; t += NT) TW[t / NK][t % NK] = et[2 * (((t / NK) * (t % NK)) % P)];
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
        for (int t = tid; t < L * NK / 2; t += NT) {
            const int f = t % L, q = t / L * 2;
            double d[2] = {0.0, 0.0}, s[2] = {0.0, 0.0};
            for (int nu = 0; nu < a.nnuc; ++nu) {
                const double2* p = reinterpret_cast<const double2*>(lines + (long long)nu * NK * P * P + line_at<NK>(q, S * f + h));
                const cd* e = mod_row(et, a, NK, nu, 2, x.i3) + q;
                const double2 dv = p[0], sv = p[NK * P / 2];
                d[0] = fma(dv.x, 2.0 * e[0].re, d[0]);
                d[1] = fma(dv.y, 2.0 * e[1].re, d[1]);
                s[0] = fma(sv.x, -2.0 * e[0].im, s[0]);
                s[1] = fma(sv.y, -2.0 * e[1].im, s[1]);
            }
            for (int i = 0; i < 2; ++i) {
                KD[f * RS + q + i] = d[i];
                KS[f * RS + q + i] = s[i];
            }
        }
        __syncthreads();
        // C: (re, im)_j = sum_i (S re_i + D im_i, S im_i - D re_i) for each row f, 16
        // outputs per work item; the 16 values D(j - i), S(j - i) of one input form windows
        // that slide down by one
        cd o[16];
        const int f = tid % L, j0 = (tid / L) * 16;
        {
            const double *kd = KD + f * RS, *ks = KS + f * RS;
            cd* row = BC + f * RS;
            double wd[16], ws[16];
            sfor<0, 16>([&](auto jc) {
                constexpr int jj = decltype(jc)::value;
                o[jj] = cd{0.0, 0.0};
                wd[jj] = kd[j0 + jj];           // windows of input i = 0
                ws[jj] = ks[j0 + jj];
            });
            sfor<0, NK>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                const cd r = row[i];
                sfor<0, 16>([&](auto jc) {
                    constexpr int jj = decltype(jc)::value;
                    o[jj].re = fma(ws[jj], r.re, fma(wd[jj], r.im, o[jj].re));
                    o[jj].im = fma(ws[jj], r.im, fma(-wd[jj], r.re, o[jj].im));
                });
                if constexpr (i + 1 < NK) {
                    // windows of input i + 1: the previous ones shifted
                    sfor<0, 15>([&](auto jc) {
                        constexpr int jj = 15 - decltype(jc)::value;
                        wd[jj] = wd[jj - 1];
                        ws[jj] = ws[jj - 1];
                    });
                    const int m = j0 - i - 1;
                    wd[0] = kd[m < 0 ? -m : m];
                    const double sv = ks[m < 0 ? -m : m];
                    ws[0] = m < 0 ? -sv : sv;
                }
            });
            __syncthreads();
            sfor<0, 16>([&](auto jc) { row[j0 + decltype(jc)::value] = o[decltype(jc)::value]; });
        }
        __syncthreads();
        // D: inverse along k2 over this residue's xi2, first NK outputs, summed over the
        // residues
        for (int j3 = tid; j3 < NK; j3 += NT) {
            cd v[32];
            sfor<0, 32>([&](auto fc) { v[decltype(fc)::value] = BC[decltype(fc)::value * RS + j3]; });
            transform<32, +1>(v);
            sfor<0, NK>([&](auto jc) {
                constexpr int j2 = decltype(jc)::value;
                const cd y = cmul(v[j2 % 32], conj(TW[h][j2]));
                ACC[j3 * RS + j2] = h == 0 ? y : cadd(ACC[j3 * RS + j2], y);
            });
        }
        __syncthreads();
    });
    for (int t = tid; t < NK * NK; t += NT) {
        const int j3 = t / NK, j2 = t % NK;
        slice[t] = ACC[j3 * RS + j2];
    }
}

// ---- E: k1 inverse, real part, written to fx.  A thread per k1 line; the result of a line
// is kept in registers (LDS at N_k = 64, whose two residues are summed).
template <typename T, int NK>
__global__ __launch_bounds__(BigShape<NK>::LE, 2) void k_thE(const fft::cd* __restrict__ W, T* __restrict__ fx,
                                                            const ThetaArgs a, unsigned t0)
{
    using namespace fft;
    using B = BigShape<NK>;
    constexpr int P = B::P, S = B::S, L = B::L, RS = B::RS, BPX = NK * NK / B::LE;
    constexpr bool REG = S == 2;
    __shared__ double TH[REG ? 1 : B::LE * RS];
    const unsigned xl = blockIdx.x / BPX;
    const int la = (int)(blockIdx.x % BPX) * B::LE + threadIdx.x;            // j3 * NK + j2
    const cd* src = W + xl * (long long)(NK * NK * NK) + la;
    T* line = fx + x_point(a, t0 + xl).xp * (NK * NK * NK) + (long long)la * NK;
    double thr[REG ? NK : 1];
    double* th = TH + (REG ? 0 : threadIdx.x * RS);
    auto at = [&](auto jc) -> double& {
        if constexpr (REG) return thr[decltype(jc)::value];
        else return th[decltype(jc)::value];
    };
    sfor<0, S / 2>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        cd v[L];
        sfor<0, L>([&](auto fc) {
            constexpr int f = decltype(fc)::value;
            v[f] = src[(long long)(L * h + f) * (NK * NK)];
        });
        transform<L, +1>(v);
        sfor<0, NK>([&](auto jc) {
            constexpr int j1 = decltype(jc)::value;
            constexpr cd m = twiddle((2 * h + 1) * j1, 2 * P, -1);
            const double t = m.im * v[j1 % L].im;
            at(jc) = fma(m.re, v[j1 % L].re, h == 0 ? t : t + at(jc));       // Re(conj(m) v)
        });
    });
    sfor<0, NK / L>([&](auto sc) {
        constexpr int k0 = decltype(sc)::value * L;
        double o[L];
        sfor<0, L>([&](auto jc) { o[decltype(jc)::value] = at(std::integral_constant<int, k0 + decltype(jc)::value>{}); });
        store_k1<T, L>(line + k0, o);
    });
}

}  // namespace chasm
