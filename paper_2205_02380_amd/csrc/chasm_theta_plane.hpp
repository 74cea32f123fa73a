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
// The factors that a lane needs for its own h (twiddles with the modulation along k2
// folded in) are held one or two to a lane and broadcast within rows of 16 lanes
// (LineFactors).
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

// o = K x for the symmetric Toeplitz matrix K[j][i] = kk[|j - i|], JB outputs at a time
// (bounds the accumulators).
template <int NK>
__device__ __forceinline__ void toeplitz_line(const double (&kk)[NK], double* line)
{
    constexpr int JB = 8;
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
// kt: the kernel values K(xi1, 2 k3 + h, 0 .. N_k - 1) of this lane's line; tw: the factors
// of this lane's half, row_j -> row_j tw_j before B and out_j -> conj(tw_j) out_j after D.
template <int NK>
__device__ __forceinline__ void plane_conv(fft::cd* slot, const double* __restrict__ kt, LineFactors<NK>& tw, int k3,
                                           int h)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    // the plane's row and the kernel values are all requested before the first use of any
    // (left to itself the compiler reads the row one value at a time)
    cd y[NK];
    cd* row = slot + k3 * S::RS;
    sfor<0, NK>([&](auto jc) { y[decltype(jc)::value] = row[decltype(jc)::value]; });
    double kk[NK];
    auto kernel_values = [&] {
        const double2* kr = reinterpret_cast<const double2*>(kt);
        sfor<0, NK / 2>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const double2 t = kr[q];
            kk[2 * q] = t.x;
            kk[2 * q + 1] = t.y;
        });
    };
    if constexpr (NK < 32) kernel_values();
    __builtin_amdgcn_sched_barrier(0);
    sfor<0, NK>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        y[j] = cmul(y[j], tw.template at<j>());
    });
    tw.renew();
    transform<NK, -1>(y);
    // at N_k = 32 the line alone takes 128 registers: with the kernel values loaded ahead the
    // transform spilled (18^3 x 32^3, two nuclei: 13.4 ms, against 12.5 with them after it)
    if constexpr (NK >= 32) {
        __builtin_amdgcn_sched_barrier(0);
        kernel_values();
    }
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

// Factors of a half line: entry j = e2_j w^{h j}, as LineFactors for lane `lane` of the
// block (lds: N_k = 8 only, the table [h][j] with rows of 9, written by this call).
template <int NK>
__device__ __forceinline__ LineFactors<NK> half_factors(const fft::cd* et, const fft::cd* e2, int h, int lane, fft::cd* lds)
{
    using namespace fft;
    if constexpr (NK == 8) {
        const int hh = (lane / 8) & 1, j = lane % 8;
        lds[hh * 9 + j] = hh ? cmul(e2[j], et[j]) : e2[j];
        return {lds + h * 9};
    } else {
        LineFactors<NK> f;
        sfor<0, NK / 16>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int j = lane % 16 + 16 * q;
            f.v[q] = h ? cmul(e2[j], et[j]) : e2[j];
        });
        return f;
    }
}

// One x-point per block at a time (persistent over x-points), N_k^2 threads, FP64
// throughout.  The xi1 axis goes by residue: chunk r < R holds xi1 = r + R m, m < C = 8
// (R C = P), the C-point transform of line_j e^{-i phi_1 j} w^{r j} folded modulo C.  Per
// chunk:
//   A  thread (k2, k3): modulated k1 line, C-point transform        -> plane m, [k3][k2]
//   BCD  plane_conv on the C planes, 2 N_k lanes each
//   E  thread (k2, k3): C-point inverse over the planes, demodulated, into the real
//      result the thread keeps in registers (16 doubles at N_k = 16)
// The modulations are products of per-axis factors: a thread forms e^{-i phi_1 j} w^{r j}
// e^{-i phi_3 k3} for its own j = k2 and broadcasts it along its line's row of lanes, for A
// and, conjugated, for E; the k2 factor rides on the twiddles of B and D.
//
// Bound: FP64 VALU (1.35e6 lane instructions per x-point at N_k = 16, 39 % of them the
// Toeplitz products; 72 % VALU busy) beside 1.1 MB of LDS traffic per x-point.  The planes
// of a chunk take 35 KB at N_k = 16; three blocks (three waves per SIMD, 168 VGPRs) share a
// CU, and one's barriers and LDS waits hide behind the others.  The loads whose latency
// showed (the row of a plane, its kernel values, the line of the next chunk) are issued
// together ahead of their use.  Measured on 61^3 x 16^3, FP32 field: 13.9 ms; 14.7 ms with
// two chunks of 16 planes, LDS factor tables and two waves per SIMD; 22.1 ms for a form
// with the k2-transformed planes side by side in LDS (140 KB, one wave per SIMD, a barrier
// after every stage).
template <typename T, int NK>
__global__ __launch_bounds__(NK * NK, NK == 16 ? 3 : 4) void k_theta(T* __restrict__ fx, const double* __restrict__ kt,
                                                                    const fft::cd* __restrict__ et, const ThetaArgs a,
                                                                    long long total)
{
    using namespace fft;
    using S = PlaneShape<NK>;
    constexpr int NT = NK * NK, P = S::P, RS = S::RS, C = 8, R = P / C;
    constexpr int GROUPS = NT / S::LANES;            // planes worked on at a time
    static_assert(C % GROUPS == 0, "whole rounds");
    constexpr bool TAB = NK == 8;                    // factors through LDS (see LineFactors)
    __shared__ cd W[C * S::SLOT];
    __shared__ cd TW[TAB ? 2 * 9 : 1], E02[TAB ? NK * 9 : 1];

    const int tid = threadIdx.x;
    const int c2 = tid % NK, c3 = tid / NK;          // k1 line (k2, k3) of stages A and E
    const int k3 = tid % NK, h = (tid / NK) & 1, grp = tid / S::LANES;
    const cd wj = et[c2];                            // w^j, j = c2

    for (long long xp = blockIdx.x; xp < total; xp += gridDim.x) {
        T* line = fx + xp * (long long)(NK * NK * NK) + tid * NK;
        double th[NK];
        sfor<0, NK>([&](auto jc) { th[decltype(jc)::value] = 0.0; });
        T fv[NK];
        load_raw<T, NK>(line, fv);

        for (int nu = 0; nu < a.nnuc; ++nu) {
            const ModRows e = mod_rows_at<NK>(et, a, xp, nu);
            const double w = a.wgt[nu];
            if constexpr (TAB) __syncthreads();      // the previous pass no longer reads the tables
            LineFactors<NK> tw = half_factors<NK>(et, e.e2, h, tid, TW);
            cd m02 = cmul(e.e1[c2], e.e3[c3]);       // entry j = c2 of this line's factors
#pragma unroll 1
            for (int r = 0; r < R; ++r) {
                LineFactors<NK> lf;
                if constexpr (TAB) {
                    E02[c3 * 9 + c2] = m02;
                    lf.v = E02 + c3 * 9;
                    __syncthreads();
                } else {
                    lf.v[0] = m02;
                }
                {   // A
                    cd y[C];
                    sfor<0, NK>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const cd m = lf.template at<j>();
                        const double f = (double)fv[j];
                        if constexpr (j < C) y[j] = cd{m.re * f, m.im * f};
                        else y[j % C] = cd{fma(m.re, f, y[j % C].re), fma(m.im, f, y[j % C].im)};
                    });
                    transform<C, -1>(y);
                    sfor<0, C>([&](auto mc) {
                        constexpr int m = decltype(mc)::value;
                        W[m * S::SLOT + c3 * RS + c2] = y[m];
                    });
                }
                __syncthreads();
#pragma unroll 1
                for (int m = grp; m < C; m += GROUPS)   // B, C, D: xi1 = r + R m, xi2 = 2 k3 + h
                    plane_conv<NK>(W + m * S::SLOT, kt + ((long long)(r + R * m) * P + 2 * k3 + h) * NK, tw, k3, h);
                __syncthreads();
                // the weight rides on E's factors; m02 moves on to the next chunk
                if constexpr (!TAB) lf.v[0] = cd{w * m02.re, w * m02.im};
                lf.renew();
                m02 = cmul(m02, wj);
                {   // E
                    load_raw<T, NK>(line, fv);       // for the next chunk's A, ahead of its first use
                    __builtin_amdgcn_sched_barrier(0);
                    cd y[C];
                    sfor<0, C>([&](auto mc) {
                        constexpr int m = decltype(mc)::value;
                        y[m] = W[m * S::SLOT + c3 * RS + c2];
                    });
                    transform<C, +1>(y);
                    if constexpr (TAB) sfor<0, C>([&](auto mc) {
                        y[decltype(mc)::value].re *= w;
                        y[decltype(mc)::value].im *= w;
                    });
                    sfor<0, NK>([&](auto jc) {
                        constexpr int j = decltype(jc)::value;
                        const cd m = lf.template at<j>();
                        th[j] = fma(m.re, y[j % C].im, fma(-m.im, y[j % C].re, th[j]));   // Im(conj(m) y)
                    });
                }
                if constexpr (TAB) __syncthreads();  // E02 is rewritten
            }
        }
        store_k1<T, NK>(line, th);
    }
}

}  // namespace chasm
