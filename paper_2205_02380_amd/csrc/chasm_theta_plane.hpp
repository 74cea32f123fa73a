// chasm_theta_plane.hpp -- the (k2, k3) part of the convolution of Theta_V on one
// (x, xi1) plane by 2 N_k lanes of one wave, and the one-block kernel built on it
// (N_k = 8 and 16).  Mathematics and notation as in chasm_theta.hpp.
//
// A plane is N_k rows (k3) of N_k complex values (k2).  Its work is
//   B  per row: k2 forward transform, zero-padded to P = 2 N_k outputs xi2 = 2 f + h:
//      the N_k-point transform of row_j w^{h j}, h = 0, 1;
//   C  per xi2: the even and the odd N_k x N_k real Toeplitz matrix along k3;
//   D  per row: k2 inverse, first N_k outputs: the sum over h of the N_k-point inverse of
//      the xi2 = 2 f + h inputs times w^{-h j}.
// Lane (h, k3) does B and D of row k3 for its h, and C of line xi2 = 2 k3 + h, so all
// 2 N_k lanes are busy in every stage with one N_k-point line each (2 N_k VGPR pairs).
// Only lanes of one wave share a plane, so nothing but the two transposes between rows
// and lines orders them: those go through the plane's own LDS slot, real parts and then
// imaginary parts, 2 N_k lines of N_k doubles -- exactly the slot's size.  The sum over h
// exchanges half of each line with the partner lane, after which each lane holds N_k/2
// outputs of its row.  The factors w^{h j} of a lane's own h are held one or two to a lane
// and broadcast within rows of 16 lanes (LineFactors).
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

// x of lane N of this lane's row of 16 lanes (a DPP move, no LDS).
template <int N>
__device__ __forceinline__ double row_bcast(double x)
{
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + N, 0xF, 0xF, true);
}

// The N_k complex factors of a line, the same for all lanes of a row of 16: lane l holds
// entries l % 16 + 16 q and every use broadcasts one (two moves; an LDS table costs a
// 16-byte read of every lane).  N_k = 8 has two lines to a row of 16 lanes and reads an
// LDS table.
template <int NK>
struct LineFactors {
    fft::cd v[NK / 16];
    template <int J>
    __device__ __forceinline__ fft::cd at() const
    {
        return {row_bcast<J % 16>(v[J / 16].re), row_bcast<J % 16>(v[J / 16].im)};
    }
    // Between two uses of the line: the broadcasts of the first are not kept for the second
    // (64 registers at N_k = 16).
    __device__ __forceinline__ void renew()
    {
        fft::sfor<0, NK / 16>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            asm volatile("" : "+v"(v[q].re), "+v"(v[q].im));
        });
    }
};
template <>
struct LineFactors<8> {
    const fft::cd* v;
    template <int J>
    __device__ __forceinline__ fft::cd at() const { return v[J]; }
    __device__ __forceinline__ void renew() {}
};

// The kernel of a line (xi1, xi2) at an x-point: of each nucleus the lane's table line
// (chasm_theta_table.hpp), and the x-point's row e^{-i phi_3 q}, the same for all lanes.
struct KernelLine {
    const double* tab;
    long long tab_nu;            // from one nucleus to the next
    const fft::cd* e3;
    long long e3_nu;
    int nnuc;
};

// D and S of nucleus nu.
template <int NK>
__device__ __forceinline__ void load_kernel(const KernelLine& kl, int nu, double (&D)[NK], double (&S)[NK])
{
    const double2* p = reinterpret_cast<const double2*>(kl.tab + nu * kl.tab_nu);
    fft::sfor<0, NK / 2>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const double2 d = p[q * 2 * NK], s = p[(q + NK / 2) * 2 * NK];
        D[2 * q] = d.x;
        D[2 * q + 1] = d.y;
        S[2 * q] = s.x;
        S[2 * q + 1] = s.y;
    });
}

// From D and S of the first nucleus, D(q) = sum_a D_a cos(phi_3 q), S(q) = sum_a S_a sin(phi_3 q).
template <int NK>
__device__ __forceinline__ void kernel_values(const KernelLine& kl, double (&D)[NK], double (&S)[NK])
{
    using namespace fft;
    sfor<0, NK>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const cd e = kl.e3[q];
        D[q] *= e.re;
        S[q] *= -e.im;
    });
#pragma unroll 1
    for (int nu = 1; nu < kl.nnuc; ++nu) {
        double d[NK], s[NK];
        load_kernel<NK>(kl, nu, d, s);
        const cd* e3 = kl.e3 + nu * kl.e3_nu;
        sfor<0, NK>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const cd e = e3[q];
            D[q] = fma(d[q], e.re, D[q]);
            S[q] = fma(s[q], -e.im, S[q]);
        });
    }
}

// (gr, gi) <- 2 (S gr + D gi, S gi - D gr), D the even and S the odd Toeplitz matrix of the
// given values.  With J the reversal, J D J = D and J S J = -S: on the even and odd parts
// e_i = x_i + x_{N-1-i}, o_i = x_i - x_{N-1-i}, i < N/2, D is one N/2 x N/2 matrix each, of
// entries D(j - i) +- D(N-1-i-j), and S carries o to e and e to o with S(j - i) +- S(N-1-i-j).
// That is half the products; the entries serve both parts of the line, and by symmetry
// the two of (i, j) and (j, i): 0.70 of the operations of four full products at N = 16.
template <int N>
__device__ __forceinline__ void toeplitz_line(const double (&D)[N], const double (&S)[N], double (&gr)[N], double (&gi)[N])
{
    using namespace fft;
    constexpr int H = N / 2;
    auto butterfly = [](double (&g)[N]) {
        sfor<0, H>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const double a = g[i], b = g[N - 1 - i];
            g[i] = a + b;
            g[N - 1 - i] = a - b;
        });
    };
    butterfly(gr);
    butterfly(gi);
    double re[N], im[N];
    sfor<0, N>([&](auto ic) { re[decltype(ic)::value] = im[decltype(ic)::value] = 0.0; });
    // the even part of output j is in [j], its odd part in [N - 1 - j]
    constexpr int B = H < 8 ? H : 8;     // tiles of B x B entries: fewer registers live at a time
    sfor<0, H * H>([&](auto tc) {
        constexpr int t = decltype(tc)::value, tile = t / (B * B), in = t % (B * B);
        constexpr int j = tile / (H / B) * B + in / B, i = tile % (H / B) * B + in % B;
        if constexpr (i <= j) {
            const std::integral_constant<int, j> jc;
            const std::integral_constant<int, i> ic;
            constexpr int d = j - i, c = N - 1 - i - j;
            const double p = D[d] + D[c], m = D[d] - D[c];
            auto even = [&](auto oc, auto nc) {
                constexpr int o = decltype(oc)::value, n = decltype(nc)::value;
                re[o] = fma(p, gi[n], re[o]);
                im[o] = fma(-p, gr[n], im[o]);
                re[N - 1 - o] = fma(m, gi[N - 1 - n], re[N - 1 - o]);
                im[N - 1 - o] = fma(-m, gr[N - 1 - n], im[N - 1 - o]);
            };
            auto odd = [&](double sp, double sm, auto oc, auto nc) {
                constexpr int o = decltype(oc)::value, n = decltype(nc)::value;
                re[o] = fma(sp, gr[N - 1 - n], re[o]);
                im[o] = fma(sp, gi[N - 1 - n], im[o]);
                re[N - 1 - o] = fma(sm, gr[n], re[N - 1 - o]);
                im[N - 1 - o] = fma(sm, gi[n], im[N - 1 - o]);
            };
            even(jc, ic);
            if constexpr (d > 0) {
                even(ic, jc);
                const double sp = S[d] + S[c], sm = S[d] - S[c];
                odd(sp, sm, jc, ic);
                odd(-sm, -sp, ic, jc);
            } else {
                odd(S[c], -S[c], jc, ic);
            }
        }
    });
    sfor<0, H>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        gr[j] = re[j] + re[N - 1 - j];
        gr[N - 1 - j] = re[j] - re[N - 1 - j];
        gi[j] = im[j] + im[N - 1 - j];
        gi[N - 1 - j] = im[j] - im[N - 1 - j];
    });
}

// Stages B, C, D of the plane in `slot`, in place.  k3, h: this lane's row and half;
// kl: the kernel of this lane's line xi2 = 2 k3 + h; tw: the factors w^{h j} of this lane's
// half.
template <int NK>
__device__ __forceinline__ void plane_conv(fft::cd* slot, const KernelLine& kl, LineFactors<NK>& tw, int k3, int h)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    cd* row = slot + k3 * S::RS;
    double gr[NK], gi[NK];
    double* col = reinterpret_cast<double*>(slot) + h * NK * S::RS + k3;      // row k3 of half h: stride RS
    double* line = reinterpret_cast<double*>(slot) + (h * NK + k3) * S::RS;   // line xi2 = 2 k3 + h
    double kd[NK], ks[NK];
    {
        cd y[NK];
        // requested before the first use of any (left to itself the compiler reads the row
        // one value at a time)
        sfor<0, NK>([&](auto jc) { y[decltype(jc)::value] = row[decltype(jc)::value]; });
        load_kernel<NK>(kl, 0, kd, ks);
        __builtin_amdgcn_sched_barrier(0);
        sfor<0, NK>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            y[j] = cmul(y[j], tw.template at<j>());
        });
        tw.renew();
        transform<NK, -1>(y);
        wave_order();
        sfor<0, NK>([&](auto fc) { col[decltype(fc)::value * S::RS] = y[decltype(fc)::value].re; });
        wave_order();
        sfor<0, NK>([&](auto ic) { gr[decltype(ic)::value] = line[decltype(ic)::value]; });
        wave_order();
        sfor<0, NK>([&](auto fc) { col[decltype(fc)::value * S::RS] = y[decltype(fc)::value].im; });
        wave_order();
        sfor<0, NK>([&](auto ic) { gi[decltype(ic)::value] = line[decltype(ic)::value]; });
    }
    kernel_values<NK>(kl, kd, ks);
    toeplitz_line<NK>(kd, ks, gr, gi);
    cd y[NK];
    wave_order();
    sfor<0, NK>([&](auto ic) { line[decltype(ic)::value] = gr[decltype(ic)::value]; });
    wave_order();
    sfor<0, NK>([&](auto fc) { y[decltype(fc)::value].re = col[decltype(fc)::value * S::RS]; });
    wave_order();
    sfor<0, NK>([&](auto ic) { line[decltype(ic)::value] = gi[decltype(ic)::value]; });
    wave_order();
    sfor<0, NK>([&](auto fc) { y[decltype(fc)::value].im = col[decltype(fc)::value * S::RS]; });
    wave_order();
    transform<NK, +1>(y);
    tw.renew();
    sfor<0, NK>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        y[j] = cmul(y[j], conj(tw.template at<j>()));
    });
    constexpr int H = NK / 2;
    sfor<0, H>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        row[h * H + j] = cd{pair_sum<NK>(y[j].re, y[j + H].re, h), pair_sum<NK>(y[j].im, y[j + H].im, h)};
    });
}

// The factors w^{h j} of a half line, as LineFactors for lane `lane` of the block (lds:
// N_k = 8 only, the table [h][j] with rows of 9, written by this call).
template <int NK>
__device__ __forceinline__ LineFactors<NK> half_factors(const fft::cd* et, int h, int lane, fft::cd* lds)
{
    using namespace fft;
    if constexpr (NK == 8) {
        const int hh = (lane / 8) & 1, j = lane % 8;
        lds[hh * 9 + j] = hh ? et[2 * j] : cd{1.0, 0.0};
        return {lds + h * 9};
    } else {
        LineFactors<NK> f;
        sfor<0, NK / 16>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            f.v[q] = h ? et[2 * (lane % 16 + 16 * q)] : cd{1.0, 0.0};
        });
        return f;
    }
}

// One x-point per block at a time (persistent over the x-points t0 .. t0 + count, whose
// first pair is p0), N_k^2 threads, FP64 throughout:
//   A  thread (k2, k3): k1 line times e^{-2 pi i j / (4 N_k)}, N_k-point transform: plane c
//      is xi1 = 2 c + 1/2                                    -> plane c, [k3][k2]
//   BCD  plane_conv on the N_k planes, 2 N_k lanes each
//   E  thread (k2, k3): N_k-point inverse over the planes; the real part, demodulated.
// Each XCD takes a contiguous share of the x-points, so that the points of a pair find its
// table lines (131 KB at N_k = 16) in one L2.
// Bound: FP64 VALU (69 % busy at N_k = 16) beside 0.6 MB of LDS traffic per x-point; two
// waves per SIMD with 233 registers, all planes of an x-point in LDS (70 KB), so that two
// barriers separate the stages.  Measured on 61^3 x 16^3, FP32 field, one nucleus: 7.7 ms
// (and 0.2 of tables); 13.9 ms for full complex spectra of the modulated field, which has
// twice the planes, a modulation on every line and one pass per nucleus.
template <typename T, int NK>
__global__ __launch_bounds__(NK * NK, NK == 16 ? 2 : 3) void k_theta(T* __restrict__ fx, const double* __restrict__ tab,
                                                                    const fft::cd* __restrict__ et, const ThetaArgs a,
                                                                    unsigned t0, unsigned count, unsigned p0)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    constexpr int NT = NK * NK, P = S::P, RS = S::RS;
    constexpr int GROUPS = NT / S::LANES;            // planes worked on at a time
    static_assert(NK % GROUPS == 0, "whole rounds");
    __shared__ cd W[NK * S::SLOT];
    __shared__ cd TW[NK == 8 ? 2 * 9 : 1];

    const int tid = threadIdx.x;
    const int c2 = tid % NK, c3 = tid / NK;          // k1 line (k2, k3) of stages A and E
    const int k3 = tid % NK, h = (tid / NK) & 1, grp = tid / S::LANES;
    LineFactors<NK> tw = half_factors<NK>(et, h, tid, TW);

    const unsigned nshare = gridDim.x % 8 ? 1 : 8, share = blockIdx.x % nshare;
    const unsigned first = (unsigned)((unsigned long long)count * share / nshare) + blockIdx.x / nshare;
    const unsigned end = (unsigned)((unsigned long long)count * (share + 1) / nshare), step = gridDim.x / nshare;
    auto line_of = [&](const XPoint& x) { return fx + x.xp * (long long)(NK * NK * NK) + tid * NK; };
    if (first >= end) return;
    XPoint x = x_point(a, t0 + first);
    T fv[NK];
    load_raw<T, NK>(line_of(x), fv);
    for (unsigned t = first; t < end; t += step) {
        T* line = line_of(x);
        KernelLine kl;
        kl.nnuc = a.nnuc;
        kl.tab = tab + ((long long)(x.pair - p0) * a.nnuc * NK * P) * P + 2 * (h * NK + k3);
        kl.tab_nu = (long long)NK * P * P;
        kl.e3 = mod_row(et, a, NK, 0, 2, x.i3);
        kl.e3_nu = (long long)(a.nx[0] + a.nx[1] + a.nx[2]) * NK;
        {   // A
            cd y[NK];
            sfor<0, NK>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                constexpr cd c = twiddle(j, 4 * NK, -1);
                const double f = (double)fv[j];
                y[j] = cd{c.re * f, c.im * f};
            });
            transform<NK, -1>(y);
            sfor<0, NK>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                W[m * S::SLOT + c3 * RS + c2] = y[m];
            });
        }
        // the next point's line, ahead of its first use
        if (t + step < end) {
            x = x_point(a, t0 + t + step);
            load_raw<T, NK>(line_of(x), fv);
        }
        __syncthreads();
#pragma unroll 1
        for (int m = grp; m < NK; m += GROUPS) {     // B, C, D: line xi2 = 2 k3 + h
            KernelLine km = kl;
            km.tab += (long long)m * (P * P);
            plane_conv<NK>(W + m * S::SLOT, km, tw, k3, h);
        }
        __syncthreads();
        {   // E
            cd y[NK];
            sfor<0, NK>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                y[m] = W[m * S::SLOT + c3 * RS + c2];
            });
            transform<NK, +1>(y);
            double th[NK];
            sfor<0, NK>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                constexpr cd c = twiddle(j, 4 * NK, -1);
                th[j] = fma(c.re, y[j].re, c.im * y[j].im);      // Re(conj(c) y)
            });
            store_k1<T, NK>(line, th);
        }
    }
}

}  // namespace chasm
