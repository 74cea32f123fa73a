// chasm_ho2d.hip -- the 2-D harmonic-oscillator workload of Sec. 5.1 (see
// include/chasm_ho2d.h): LPC1 with the patched-spline characteristic step in x and the
// spectral k-derivative Theta[f] = omega x d_k f, all FP64.
//
// Transform path (nk a power of two in 64..1024): a step is two launches, and the
// library's fields are kept as [x][k], so that the k transforms read contiguous lines
// and the x sweeps read short contiguous runs; k_ho_turn converts the caller's [k][x]
// field at both ends of a call.
//   k_ho_advect  the characteristic step of LB k-lines per block, lines of runtime
//                length in LDS: PMBC interface slopes (eqs. 3.4-3.5, eight lanes per dot
//                product), each patch's reduced Hermite system by the sweeping method
//                (one thread per patch and line), the Hermite ghosts, and the 4-tap
//                evaluation by the owning patch (eqs. 3.7-3.8, Sec. 3.1.3), out of place;
//                departure points outside the line give 0 unless the descriptor asks
//                for ghost extrapolation.
//   k_ho_dk      Theta by transforms, for nk = L1 L2: two real k-lines (x columns 2c,
//                2c+1) form one complex line, since the derivative F^-1 diag(i xi) F maps
//                real lines to real lines; a four-step transform (L1-point register
//                transforms over stride-L2 elements, twiddles, L2-point register
//                transforms), the multiply by i xi / nk (Nyquist mode 0) and the inverse
//                in reverse order, with two LDS transposes per line.  The corrector form
//                reads FA, GA, transforms Y = FA + tau GA, forms the new field FA + tau/2
//                (GA + Theta Y) and, unless the step is the call's last, transforms that
//                again for the next step's Theta F: the column is already in registers.
//                At nx = 241, nk = 512 a step is 17.3 us, against 28.9 us in three
//                launches on [k][x] fields.
//   k_ho_dk512   nk = 512: the same transform pair in three levels of 8-point
//                transforms, one complex line per 64-thread block.
// Dense path (any other even nk; fields [k][x]):
//   k_ho_theta   out[k][x] = omega x sum_q D[k][q] f[q][x], a dense FP64 contraction with
//                the circulant spectral differentiation matrix, 32 x 32 output tiles
//                staged through LDS, 2 x 2 outputs per thread.
//   k_ho_combine the predictor / corrector combinations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <new>
#include <string>
#include <vector>

#include "../../include/chasm_ho2d.h"
#include "chasm_fft.hpp"
#include "chasm_tables.hpp"

namespace chasm {
void set_last_error(const std::string& msg);

struct HoArgs {
    int N, M, P, mlast, g, nk, inflow;
    double hx;
    const double* stencil;     // (P+1) x (2g+1), slopes (not times h)
    const double* lu;          // inv, ainv, cp of the reduced patch system (patch_factors): the first
                               // HO_LU rows of a long patch (rows before the last do not depend on its length)
    double inv_l[2], ainv_l[2];   // last row: patches of M cells, the last patch
    const int* shift;          // nk
    const double* w;           // nk x 4
};

// LDS doubles of k_ho_advect per line: the nodes (odd row length, but for the longest
// lines), the slopes and the patches' coefficients.
__host__ __device__ constexpr int ho_row(int LB, int N) { return LB > 2 ? N | 1 : N; }
__host__ __device__ constexpr int ho_line_doubles(int LB, int N, int P) { return ho_row(LB, N) + (N - 1 + 3 * P) + (P + 1); }

// Rows of the patch factors that are kept: the recursion contracts by (2 - sqrt 3)^2 = 0.07
// a row, so from row 14 on the factors are one constant to double precision.
constexpr int HO_LU = 32;

// The lines of two stacked fields of nk x N values: line L is k node L % nk of field
// L / nk.  XK: fields are [x][k], else [k][x].  Bound by latency (a 1 MB field over 256
// blocks): every global load is issued before the first barrier, the slopes take (2 g + 1)
// / 8 terms a lane, and the serial part is one patch sweep of 2 M dependent multiply-adds
// out of LDS.  10.6 us a launch at nx = 241, 1024 lines, against
// 14.7 us for the product of each patch with its precomputed inverse.
template <int LB, bool XK>
__global__ __launch_bounds__(256) void k_ho_advect(const double* __restrict__ in, double* __restrict__ out, const HoArgs a,
                                                  int nlines)
{
    extern __shared__ double sm[];
    const int N = a.N, M = a.M, P = a.P, NS = ho_row(LB, N);
    const int ES = N - 1 + 3 * P;                    // sum over patches of (m + 3)
    double* phi = sm;                                // [LB][NS]
    double* dsl = phi + LB * NS;                     // [LB][P+1] slopes times h
    double* eta = dsl + LB * (P + 1);                // [LB][ES], patch l at l (M+3): eta_{-1..m+1}
    // the factors [inv, ainv, cp][HO_LU]: in LDS, but for the longest lines, which fill it
    double* const lds_lu = eta + LB * ES;
    const double* const lu = LB > 2 ? lds_lu : a.lu;
    const double *const inv = lu, *const ainv = lu + HO_LU, *const cp = lu + 2 * HO_LU;
    const int line0 = blockIdx.x * LB;
    const int tid = threadIdx.x, W = 2 * a.g + 1, nrow = LB * (P + 1);
    auto at = [&](int L, int j) -> long long {
        if constexpr (XK) {
            const int fld = L / a.nk, kk = L - fld * a.nk;
            return ((long long)fld * N + j) * a.nk + kk;
        } else {
            return (long long)L * N + j;
        }
    };
    // interface row e of the block's LB (P + 1): line e / (P + 1), interface e % (P + 1)
    auto iface = [&](int q) { return q < P ? q * M : N - 1; };
    constexpr int PRE = 8;                           // taps per lane fetched ahead (first 32 rows)
    double cf[PRE];
    {
        const int e = tid / 8, q = e % (P + 1);
#pragma unroll
        for (int u = 0; u < PRE; ++u) {
            const int t = tid % 8 + 8 * u;
            cf[u] = e < nrow && t < W ? a.stencil[q * W + t] : 0.0;
        }
    }
    if (LB > 2 && tid < 3 * HO_LU) lds_lu[tid] = a.lu[tid];
    // [x][k]: a thread's outputs all belong to line tid % LB
    const int my_k = (line0 + tid % LB) % a.nk;
    const int my_shift = a.shift[my_k];
    const double my_w[4] = {a.w[4 * my_k], a.w[4 * my_k + 1], a.w[4 * my_k + 2], a.w[4 * my_k + 3]};
    for (int e = tid; e < LB * N; e += 256) {
        const int ln = XK ? e % LB : e / N, j = XK ? e / LB : e - ln * N;
        phi[ln * NS + j] = line0 + ln < nlines ? in[at(line0 + ln, j)] : 0.0;
    }
    __syncthreads();
    for (int e0 = 0; e0 < nrow; e0 += 32) {          // eight lanes per interface slope
        const int e = e0 + tid / 8;
        double acc = 0.0;
        if (e < nrow) {
            const int ln = e / (P + 1), q = e % (P + 1);
            const double* v = phi + ln * NS;
            const int j0 = iface(q) - a.g;
            int t = tid % 8;
            if (e0 == 0) {
                // taps off the stencil or the line have coefficient 0 and take a node of the
                // stencil, so that a slope sees no other node, finite or not
                const int last = min(j0 + W, N) - 1;
#pragma unroll
                for (int u = 0; u < PRE; ++u) {
                    const int j = j0 + t + 8 * u;
                    acc = fma(cf[u], v[j < 0 ? 0 : (j < last ? j : last)], acc);
                }
                t += 8 * PRE;
            }
            for (; t < W; t += 8) {
                const int j = j0 + t;
                if (j >= 0 && j < N) acc = fma(a.stencil[q * W + t], v[j], acc);
            }
        }
        acc += __shfl_xor(acc, 1, 64);
        acc += __shfl_xor(acc, 2, 64);
        acc += __shfl_xor(acc, 4, 64);
        if (e < nrow && tid % 8 == 0) dsl[e] = acc * a.hx;
    }
    __syncthreads();
    // forward sweep and back substitution of one patch per thread; the LDS reads of eight
    // nodes are issued together, ahead of their part of the dependent chain
    for (int e = tid; e < LB * P; e += 256) {
        const int ln = e / P, l = e % P, last = l == P - 1;
        const int m = last ? a.mlast : M;
        const double dL = dsl[ln * (P + 1) + l], dR = dsl[ln * (P + 1) + l + 1];
        const double* v = phi + ln * NS + l * M;
        double* E = eta + ln * ES + l * (M + 3) + 1;
        const double inv_c = inv[HO_LU - 1], ainv_c = ainv[HO_LU - 1], cp_c = cp[HO_LU - 1];
        double x = fma(1.0 / 3.0, dL, v[0]) * inv[0];
        E[0] = x;
        int i = 1;
        for (; i + 8 <= m; i += 8) {                 // rows i .. i + 7
            double r[8], f[8];
            if (i + 7 < HO_LU) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    r[u] = v[i + u] * inv[i + u];
                    f[u] = ainv[i + u];
                }
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    r[u] = v[i + u] * inv_c;
                    f[u] = ainv_c;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = x = fma(-f[u], x, r[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u) E[i + u] = r[u];
        }
        for (; i < m; ++i) {
            const int k = i < HO_LU ? i : HO_LU - 1;
            E[i] = x = fma(-ainv[k], x, v[i] * inv[k]);
        }
        E[m] = x = fma(-a.ainv_l[last], x, fma(-1.0 / 3.0, dR, v[m]) * a.inv_l[last]);
        i = m - 1;
        for (; i - 7 >= 0; i -= 8) {                 // rows i .. i - 7
            double r[8], f[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = E[i - u];
            if (i < HO_LU) {
#pragma unroll
                for (int u = 0; u < 8; ++u) f[u] = cp[i - u];
            } else if (i - 7 >= HO_LU) {
#pragma unroll
                for (int u = 0; u < 8; ++u) f[u] = cp_c;
            } else {
#pragma unroll
                for (int u = 0; u < 8; ++u) f[u] = cp[i - u < HO_LU ? i - u : HO_LU - 1];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = x = fma(-f[u], x, r[u]);
#pragma unroll
            for (int u = 0; u < 8; ++u) E[i - u] = r[u];
        }
        for (; i >= 0; --i) E[i] = x = fma(-cp[i < HO_LU ? i : HO_LU - 1], x, E[i]);
        E[-1] = fma(-2.0, dL, E[1]);                              // eta_{-1} = eta_1 - 2 h d_L
        E[m + 1] = fma(2.0, dR, E[m - 1]);                        // eta_{m+1} = eta_{m-1} + 2 h d_R
    }
    __syncthreads();
    for (int e = tid; e < LB * N; e += 256) {
        const int ln = XK ? e % LB : e / N, j = XK ? e / LB : e - ln * N, L = line0 + ln;
        if (L >= nlines) continue;
        const int kk = XK ? 0 : L % a.nk;
        const int c = j + (XK ? my_shift : a.shift[kk]);         // departure cell
        double w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = XK ? my_w[r] : a.w[4 * kk + r];
        double v = 0.0;
        // departure point inside [x_0, x_{N-1}]: cell 0 .. N-2, or exactly node N-1
        // (beta = 0, i.e. w3 = beta^3/6 = 0)
        const bool inside = c >= 0 && (c < N - 1 || (c == N - 1 && w[3] == 0.0));
        if ((inside || a.inflow == 1) && c >= -4 && c <= N + 2) {
            const int l = c < 0 ? 0 : min(c / M, P - 1);         // owner patch
            const int m = l < P - 1 ? M : a.mlast;
            const int nu = c - l * M;
            const double* E = eta + ln * ES + l * (M + 3);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int u = nu - 1 + r;                        // eta_u, zero beyond the ghosts
                if (u >= -1 && u <= m + 1) v = fma(w[r], E[u + 1], v);
            }
        }
        out[at(L, j)] = v;
    }
}

// dst[c][r] = src[r][c] of a rows x cols matrix, 32 x 32 tiles through LDS.
__global__ __launch_bounds__(256) void k_ho_turn(const double* __restrict__ src, double* __restrict__ dst, int rows, int cols)
{
    __shared__ double tile[32][33];
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32, tx = threadIdx.x % 32, ty = threadIdx.x / 32;
    for (int i = ty; i < 32; i += 8)
        if (r0 + i < rows && c0 + tx < cols) tile[i][tx] = src[(long long)(r0 + i) * cols + c0 + tx];
    __syncthreads();
    for (int i = ty; i < 32; i += 8)
        if (c0 + i < cols && r0 + tx < rows) dst[(long long)(c0 + i) * rows + r0 + tx] = tile[tx][i];
}

__global__ __launch_bounds__(256) void k_ho_theta(const double* __restrict__ D, const double* __restrict__ f,
                                                 double* __restrict__ out, int nk, int nx, double x_lo, double hx,
                                                 double omega)
{
    // 32 x 32 output tile per block (2 x 2 per thread), k-chunks of 32 through LDS
    __shared__ double As[32][33];                       // As[q][r] = D[r0 + r][q0 + q]
    __shared__ double Bs[32][33];                       // Bs[q][c] = f[q0 + q][c0 + c]
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    double acc[2][2] = {};
    for (int q0 = 0; q0 < nk; q0 += 32) {
        for (int e = threadIdx.x; e < 32 * 32; e += 256) {
            const int rr = e / 32, qq = e % 32;
            const int r = r0 + rr, q = q0 + qq;
            As[qq][rr] = (r < nk && q < nk) ? D[(long long)r * nk + q] : 0.0;
            const int qb = e / 32, cc = e % 32;
            const int qf = q0 + qb, x = c0 + cc;
            Bs[qb][cc] = (qf < nk && x < nx) ? f[(long long)qf * nx + x] : 0.0;
        }
        __syncthreads();
#pragma unroll 8
        for (int qq = 0; qq < 32; ++qq) {
            const double a0 = As[qq][ty], a1 = As[qq][ty + 16];
            const double b0 = Bs[qq][tx], b1 = Bs[qq][tx + 16];
            acc[0][0] = fma(a0, b0, acc[0][0]);
            acc[0][1] = fma(a0, b1, acc[0][1]);
            acc[1][0] = fma(a1, b0, acc[1][0]);
            acc[1][1] = fma(a1, b1, acc[1][1]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 2; ++i) {
        const int r = r0 + ty + 16 * i;
        if (r >= nk) continue;
        for (int j = 0; j < 2; ++j) {
            const int x = c0 + tx + 16 * j;
            if (x < nx) out[(long long)r * nx + x] = omega * (x_lo + x * hx) * acc[i][j];
        }
    }
}

struct DkArgs {
    int nx;
    double x_lo, hx, hk, omega, tau;
};

// Complex lines per block and threads per block of k_ho_dk (one wave).
template <int L1, int L2>
struct DkShape {
    static constexpr int L = L1 * L2;
    static constexpr int TL = L2 > L1 ? L2 : L1;     // threads per complex line
    static constexpr int CLB = 64 / TL;              // complex lines per block
    static constexpr int NT = CLB * TL;
    static constexpr int RS = L2 + 1;                // LDS row of [k1][n2], padded
};

// What a k transform kernel does with its columns (fields [x][k]):
//   DK_THETA    out2 = Theta a
//   DK_LAST     out = (a + tau/2 b) + tau/2 Theta (a + tau b)
//   DK_STEP     the same out, and out2 = Theta out (the next step's first derivative)
enum DkMode { DK_THETA = 0, DK_LAST = 1, DK_STEP = 2 };

// tw[j] = e^{+2 pi i j / L}.  Index convention of the four-step transform: element
// n = L2 n1 + n2, frequency m = k1 + L1 k2.
template <int L1, int L2, int MODE>
__global__ __launch_bounds__(64) void k_ho_dk(const double* __restrict__ a, const double* __restrict__ b,
                                              double* __restrict__ out, double* __restrict__ out2,
                                              const fft::cd* __restrict__ tw, const DkArgs p)
{
    using namespace fft;
    using S = DkShape<L1, L2>;
    static_assert(S::NT == 64, "one wave per block");
    constexpr int L = S::L;
    __shared__ cd lds[S::CLB * L1 * S::RS];
    const int lt = threadIdx.x % S::TL, cl = threadIdx.x / S::TL;
    const int xa = 2 * (blockIdx.x * S::CLB + cl), xb = xa + 1;
    const bool has_a = xa < p.nx, has_b = xb < p.nx;
    cd* Y = lds + cl * L1 * S::RS;
    const bool rows = lt < L2 && has_a;              // thread n2 = lt of steps 1 and 3
    const int n2 = lt;
    const long long ca = (long long)xa * L + n2, cb = (long long)xb * L + n2;   // + L2 n1
    const double h = 0.5 * p.tau, tau = p.tau, hk = p.hk;
    const double fa = p.omega * (p.x_lo + xa * p.hx), fb = p.omega * (p.x_lo + xb * p.hx);

    // v: elements L2 n1 + n2 of the column pair -> its k derivative at the same elements
    auto derive = [&](cd (&v)[L1]) {
        // Step 1 (thread n2): L1-point transforms over n1, twiddle e^{-2 pi i n2 k1 / L}.
        if (rows) {
            transform<L1, -1>(v);
            sfor<0, L1>([&](auto kc) {
                constexpr int k1 = decltype(kc)::value;
                cd w = v[k1];
                if constexpr (k1 > 0) w = cmul(w, conj(tw[(n2 * k1) & (L - 1)]));
                Y[k1 * S::RS + n2] = w;
            });
        }
        __syncthreads();
        // Step 2 (thread k1 = lt): L2-point transforms over n2 give X[k1 + L1 k2]; multiply by
        // i xi_m / L; inverse L2-point transforms; twiddle e^{+2 pi i n2 k1 / L}.
        if (lt < L1 && has_a) {
            const int k1 = lt;
            cd u[L2];
            sfor<0, L2>([&](auto ic) { u[decltype(ic)::value] = Y[k1 * S::RS + decltype(ic)::value]; });
            transform<L2, -1>(u);
            const double unit = 2.0 * kPi / (L * hk) / L;
            sfor<0, L2>([&](auto kc) {
                constexpr int k2 = decltype(kc)::value;
                const int m = k1 + L1 * k2;
                const double xi = m < L / 2 ? (double)m * unit : (m == L / 2 ? 0.0 : (double)(m - L) * unit);
                u[k2] = {-xi * u[k2].im, xi * u[k2].re};
            });
            transform<L2, +1>(u);
            sfor<0, L2>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                cd w = u[n];
                if constexpr (n > 0) w = cmul(w, tw[(n * k1) & (L - 1)]);
                Y[k1 * S::RS + n] = w;
            });
        }
        __syncthreads();
        // Step 3 (thread n2): inverse L1-point transforms over k1 give d_k y at L2 n1 + n2;
        // real part column xa, imaginary part column xb.
        if (rows) {
            sfor<0, L1>([&](auto kc) { v[decltype(kc)::value] = Y[decltype(kc)::value * S::RS + n2]; });
            transform<L1, +1>(v);
        }
    };

    cd v[L1], keep[MODE == DK_THETA ? 1 : L1];
    if (rows) {
        sfor<0, L1>([&](auto ic) {
            constexpr int n1 = decltype(ic)::value;
            v[n1] = {a[ca + L2 * n1], has_b ? a[cb + L2 * n1] : 0.0};
            if constexpr (MODE != DK_THETA) {
                const cd y = v[n1], g = {b[ca + L2 * n1], has_b ? b[cb + L2 * n1] : 0.0};
                v[n1] = {fma(tau, g.re, y.re), fma(tau, g.im, y.im)};
                keep[n1] = {fma(h, g.re, y.re), fma(h, g.im, y.im)};
            }
        });
    }
    derive(v);
    if constexpr (MODE != DK_THETA) {
        if (rows) {
            sfor<0, L1>([&](auto ic) {
                constexpr int n1 = decltype(ic)::value;
                v[n1] = {fma(h, fa * v[n1].re, keep[n1].re), has_b ? fma(h, fb * v[n1].im, keep[n1].im) : 0.0};
                out[ca + L2 * n1] = v[n1].re;
                if (has_b) out[cb + L2 * n1] = v[n1].im;
            });
        }
    }
    if constexpr (MODE == DK_STEP) {
        __syncthreads();   // step 3 has read the rows that step 1 writes
        derive(v);
    }
    if constexpr (MODE != DK_LAST) {
        if (rows) {
            sfor<0, L1>([&](auto ic) {
                constexpr int n1 = decltype(ic)::value;
                out2[ca + L2 * n1] = fa * v[n1].re;
                if (has_b) out2[cb + L2 * n1] = fb * v[n1].im;
            });
        }
    }
}

// nk = 512 = 8 x 8 x 8: a three-level form of the same transform pair, so that every
// thread's serial chain is six 8-point transforms (the four-step form above runs two
// 32-point transforms per thread in its middle step).  One complex line (x columns 2c,
// 2c+1) per 64-thread block.  Index convention: element n = 64 n1 + 8 n2 + n3,
// frequency m = m1 + 8 m2 + 64 m3;
//   step 1   (n2, n3): 8-point transform over n1, twiddle e^{-2 pi i (8 n2 + n3) m1 / 512}
//   step 2   (m1, n3): 8-point transform over n2, twiddle e^{-2 pi i 8 n3 m2 / 512}
//   step 3   (m1, m2): 8-point transform over n3, times i xi_m / 512, inverse over m3
//   steps 2', 1': the inverses of steps 2 and 1 with conjugate twiddles.
// Thread (n2, n3) = (t / 8, t % 8) in step 1, so a wave's accesses are contiguous.
template <int MODE>
__global__ __launch_bounds__(64) void k_ho_dk512(const double* __restrict__ a, const double* __restrict__ b,
                                                double* __restrict__ out, double* __restrict__ out2,
                                                const fft::cd* __restrict__ tw, const DkArgs p)
{
    using namespace fft;
    constexpr int L = 512, RS = 66;                 // LDS rows of 64 values, padded
    __shared__ cd S1[8 * RS];                        // [m1][n2][n3]
    __shared__ cd S2[8 * RS];                        // [m1][m2][n3]
    const int t = threadIdx.x, lo = t & 7, hi = t >> 3;
    const int xa = 2 * blockIdx.x, xb = xa + 1;
    const bool has_b = xb < p.nx;
    const double h = 0.5 * p.tau, tau = p.tau, hk = p.hk;
    const double fa = p.omega * (p.x_lo + xa * p.hx), fb = p.omega * (p.x_lo + xb * p.hx);
    const long long ca = (long long)xa * L + t, cb = (long long)xb * L + t;     // + 64 n1
    // twiddles of this thread's elements, used forward (conjugated) and inverse
    cd w1[8], w2[8];
    sfor<1, 8>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        w1[m] = tw[(t * m) & (L - 1)];
        w2[m] = tw[(8 * hi * m) & (L - 1)];
    });

    // v: elements 64 n1 + t of the column pair -> its k derivative at the same elements
    auto derive = [&](cd (&v)[8]) {
        // step 1: (n2, n3) = (hi, lo)
        transform<8, -1>(v);
        sfor<0, 8>([&](auto mc) {
            constexpr int m1 = decltype(mc)::value;
            S1[m1 * RS + t] = m1 > 0 ? cmul(v[m1], conj(w1[m1])) : v[m1];
        });
        __syncthreads();
        // step 2: (m1, n3) = (lo, hi)
        sfor<0, 8>([&](auto ic) { v[decltype(ic)::value] = S1[lo * RS + 8 * decltype(ic)::value + hi]; });
        transform<8, -1>(v);
        sfor<0, 8>([&](auto mc) {
            constexpr int m2 = decltype(mc)::value;
            S2[lo * RS + 8 * m2 + hi] = m2 > 0 ? cmul(v[m2], conj(w2[m2])) : v[m2];
        });
        __syncthreads();
        // step 3: (m1, m2) = (lo, hi); the row is this thread's alone, read and written back
        sfor<0, 8>([&](auto ic) { v[decltype(ic)::value] = S2[lo * RS + 8 * hi + decltype(ic)::value]; });
        transform<8, -1>(v);
        const double unit = 2.0 * kPi / (L * hk) / L;
        sfor<0, 8>([&](auto mc) {
            constexpr int m3 = decltype(mc)::value;
            const int m = lo + 8 * hi + 64 * m3;
            const double xi = m < L / 2 ? (double)m * unit : (m == L / 2 ? 0.0 : (double)(m - L) * unit);
            v[m3] = {-xi * v[m3].im, xi * v[m3].re};
        });
        transform<8, +1>(v);
        sfor<0, 8>([&](auto ic) { S2[lo * RS + 8 * hi + decltype(ic)::value] = v[decltype(ic)::value]; });
        __syncthreads();
        // step 2': (m1, n3) = (lo, hi)
        sfor<0, 8>([&](auto mc) {
            constexpr int m2 = decltype(mc)::value;
            const cd x = S2[lo * RS + 8 * m2 + hi];
            v[m2] = m2 > 0 ? cmul(x, w2[m2]) : x;
        });
        transform<8, +1>(v);
        sfor<0, 8>([&](auto ic) { S1[lo * RS + 8 * decltype(ic)::value + hi] = v[decltype(ic)::value]; });
        __syncthreads();
        // step 1': (n2, n3) = (hi, lo); d_k y at elements 64 n1 + 8 n2 + n3
        sfor<0, 8>([&](auto mc) {
            constexpr int m1 = decltype(mc)::value;
            const cd x = S1[m1 * RS + t];
            v[m1] = m1 > 0 ? cmul(x, w1[m1]) : x;
        });
        transform<8, +1>(v);
    };

    cd v[8], keep[MODE == DK_THETA ? 1 : 8];
    sfor<0, 8>([&](auto ic) {
        constexpr int n1 = decltype(ic)::value;
        v[n1] = {a[ca + 64 * n1], has_b ? a[cb + 64 * n1] : 0.0};
        if constexpr (MODE != DK_THETA) {
            const cd y = v[n1], g = {b[ca + 64 * n1], has_b ? b[cb + 64 * n1] : 0.0};
            v[n1] = {fma(tau, g.re, y.re), fma(tau, g.im, y.im)};
            keep[n1] = {fma(h, g.re, y.re), fma(h, g.im, y.im)};
        }
    });
    derive(v);
    if constexpr (MODE != DK_THETA) {
        sfor<0, 8>([&](auto ic) {
            constexpr int n1 = decltype(ic)::value;
            v[n1] = {fma(h, fa * v[n1].re, keep[n1].re), has_b ? fma(h, fb * v[n1].im, keep[n1].im) : 0.0};
            out[ca + 64 * n1] = v[n1].re;
            if (has_b) out[cb + 64 * n1] = v[n1].im;
        });
    }
    if constexpr (MODE == DK_STEP) derive(v);   // step 1 writes S1 entries this thread alone has just read
    if constexpr (MODE != DK_LAST) {
        sfor<0, 8>([&](auto ic) {
            constexpr int n1 = decltype(ic)::value;
            out2[ca + 64 * n1] = fa * v[n1].re;
            if (has_b) out2[cb + 64 * n1] = fb * v[n1].im;
        });
    }
}

// mode 0: dst = a + c b;  mode 1: dst = a + c (b + y)
__global__ __launch_bounds__(256) void k_ho_combine(double* __restrict__ dst, const double* __restrict__ a,
                                                   const double* __restrict__ b, const double* __restrict__ y,
                                                   long long n, double c, int mode)
{
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
        dst[i] = mode == 0 ? fma(c, b[i], a[i]) : fma(c, b[i] + y[i], a[i]);
}

// Spectral differentiation on the periodic grid of n (even) points, spacing h:
// D[p][q] = d(p - q), d(0) = 0, d(r) = (pi / (n h)) (-1)^r cot(pi r / n) -- the matrix of
// F^-1 diag(i xi) F with the Nyquist mode's derivative set to zero.
static std::vector<double> spectral_dk(int n, double h)
{
    std::vector<double> d(n, 0.0), D((size_t)n * n);
    for (int r = 1; r < n; ++r) d[r] = (M_PI / (n * h)) * ((r % 2) ? -1.0 : 1.0) / std::tan(M_PI * r / n);
    for (int p = 0; p < n; ++p)
        for (int q = 0; q < n; ++q) D[(size_t)p * n + q] = d[((p - q) % n + n) % n];
    return D;
}

}  // namespace chasm

using namespace chasm;

struct chasm_ho2d_s {
    chasm_ho2d_desc desc;
    hipStream_t stream = nullptr;
    HoArgs args{};
    void* tables = nullptr;
    double* D = nullptr;             // dense path: the differentiation matrix
    fft::cd* tw = nullptr;           // transform path: e^{+2 pi i j / nk}, j < nk
    double *X = nullptr, *XA = nullptr;   // two fields each
    double *Y = nullptr, *Z = nullptr;    // dense path: the predictor and its derivative
    double* f = nullptr;
    long long n = 0;
    bool poisoned = false;
};

static chasm_status hfail(chasm_status st, const std::string& m)
{
    set_last_error(m);
    return st;
}

// Transform path for nk in {64, ..., 1024}: nk = L1 L2.
static bool dk_by_transform(int nk) { return nk >= 64 && nk <= 1024 && (nk & (nk - 1)) == 0; }

template <int L1, int L2>
static void launch_dk_t(int mode, const double* a, const double* b, double* out, double* out2, const fft::cd* tw,
                        const DkArgs& p, hipStream_t s)
{
    using S = DkShape<L1, L2>;
    const int ncl = (p.nx + 1) / 2;
    const dim3 grid((unsigned)((ncl + S::CLB - 1) / S::CLB));
    auto k = mode == DK_THETA ? k_ho_dk<L1, L2, DK_THETA> : mode == DK_LAST ? k_ho_dk<L1, L2, DK_LAST> : k_ho_dk<L1, L2, DK_STEP>;
    hipLaunchKernelGGL(k, grid, dim3(S::NT), 0, s, a, b, out, out2, tw, p);
}

static void launch_dk(int nk, int mode, const double* a, const double* b, double* out, double* out2, const fft::cd* tw,
                      const DkArgs& p, hipStream_t s)
{
    switch (nk) {
    case 64: launch_dk_t<8, 8>(mode, a, b, out, out2, tw, p, s); break;
    case 128: launch_dk_t<8, 16>(mode, a, b, out, out2, tw, p, s); break;
    case 256: launch_dk_t<16, 16>(mode, a, b, out, out2, tw, p, s); break;
    case 512: {
        auto k = mode == DK_THETA ? k_ho_dk512<DK_THETA> : mode == DK_LAST ? k_ho_dk512<DK_LAST> : k_ho_dk512<DK_STEP>;
        hipLaunchKernelGGL(k, dim3((unsigned)((p.nx + 1) / 2)), dim3(64), 0, s, a, b, out, out2, tw, p);
        break;
    }
    default: launch_dk_t<32, 32>(mode, a, b, out, out2, tw, p, s); break;
    }
}

// Four lines per block where they fit in 64 KB of LDS (256 blocks at nk = 512), else two
// (every accepted line fits: see the limit in chasm_ho2d_create).
template <bool XK>
static void launch_advect(const double* in, double* out, const HoArgs& a, hipStream_t s)
{
    const int nlines = 2 * a.nk;
    const size_t lds4 = (4 * (size_t)ho_line_doubles(4, a.N, a.P) + 3 * HO_LU) * sizeof(double);
    const size_t lds2 = 2 * (size_t)ho_line_doubles(2, a.N, a.P) * sizeof(double);
    if (lds4 <= 65536)
        hipLaunchKernelGGL((k_ho_advect<4, XK>), dim3((unsigned)((nlines + 3) / 4)), dim3(256), lds4, s, in, out, a, nlines);
    else
        hipLaunchKernelGGL((k_ho_advect<2, XK>), dim3((unsigned)((nlines + 1) / 2)), dim3(256), lds2, s, in, out, a, nlines);
}

extern "C" {

chasm_status chasm_ho2d_create(const chasm_ho2d_desc* d, void* f_dev, void* hip_stream, chasm_ho2d_t* out)
{
    if (!out) return hfail(CHASM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!d || !f_dev) return hfail(CHASM_EINVAL, "NULL argument");
    if (d->nx < 2 || d->nx > 1024) return hfail(CHASM_EINVAL, "nx must be in 2..1024");
    if (d->nk < 2 || d->nk > 4096 || d->nk % 2) return hfail(CHASM_EINVAL, "nk must be even, 2..4096");
    if (!(d->hx > 0) || !(d->hk > 0) || !std::isfinite(d->x_lo) || !std::isfinite(d->k_lo) || !std::isfinite(d->hx) ||
        !std::isfinite(d->hk))
        return hfail(CHASM_EINVAL, "grid spacings must be finite and > 0");
    if (d->patch < 2 || d->patch > d->nx - 1) return hfail(CHASM_EINVAL, "patch must be in 2..nx-1");
    if (d->ghost < 1 || d->ghost > d->nx - 1) return hfail(CHASM_EINVAL, "ghost must be in 1..nx-1");
    if (!std::isfinite(d->omega) || !(d->tau > 0) || !std::isfinite(d->tau))
        return hfail(CHASM_EINVAL, "omega must be finite and tau finite and > 0");
    if (d->inflow != 0 && d->inflow != 1) return hfail(CHASM_EINVAL, "inflow must be 0 or 1");

    AxisTables at;
    std::string err;
    if (!build_axis_tables(d->nx, d->patch, d->ghost, d->ghost, d->hx, 0, d->nk, d->k_lo, d->hk, d->tau, at, err))
        return hfail(CHASM_EINVAL, err);
    const int P = at.P, M = d->patch, mlast = at.MLAST;
    if ((size_t)2 * (2 * d->nx + 4 * P) * sizeof(double) > 65536)
        return hfail(CHASM_EINVAL, "lines too long for the LDS line kernel (2 lines of 2 nx + 4 P doubles <= 64 KiB)");
    const bool by_transform = dk_by_transform(d->nk);
    std::vector<double> LU((size_t)3 * (HO_LU + 1)), LM((size_t)3 * (M + 1)), LL((size_t)3 * (mlast + 1));
    patch_factors(HO_LU, LU.data(), LU.data() + (HO_LU + 1), LU.data() + 2 * (HO_LU + 1));
    for (int i = 1; i < 3; ++i) std::copy_n(LU.begin() + i * (HO_LU + 1), HO_LU, LU.begin() + i * HO_LU);
    LU.resize((size_t)3 * HO_LU);
    patch_factors(M, LM.data(), LM.data() + (M + 1), LM.data() + 2 * (M + 1));
    patch_factors(mlast, LL.data(), LL.data() + (mlast + 1), LL.data() + 2 * (mlast + 1));
    const std::vector<double> D = by_transform ? std::vector<double>() : spectral_dk(d->nk, d->hk);
    std::vector<fft::cd> TW;
    if (by_transform)
        for (int j = 0; j < d->nk; ++j) TW.push_back(fft::twiddle(j, d->nk, +1));

    chasm_ho2d_s* h = new (std::nothrow) chasm_ho2d_s();
    if (!h) return hfail(CHASM_ENOMEM, "host allocation failed");
    h->desc = *d;
    h->stream = (hipStream_t)hip_stream;
    h->f = static_cast<double*>(f_dev);
    h->n = (long long)d->nk * d->nx;
    auto bail = [&](chasm_status s, const std::string& m) {
        chasm_ho2d_destroy(h);
        (void)hipGetLastError();   // reported by this call, not by the next launch of another handle
        return hfail(s, m);
    };
    // one block: stencil | patch factors | w (doubles), then shift (ints)
    const size_t nd = at.stencil.size() + LU.size() + at.w.size();
    std::vector<char> blob(nd * sizeof(double) + at.shift.size() * sizeof(int));
    double* dp = reinterpret_cast<double*>(blob.data());
    size_t o = 0;
    const size_t o_st = o; std::copy(at.stencil.begin(), at.stencil.end(), dp + o); o += at.stencil.size();
    const size_t o_lu = o; std::copy(LU.begin(), LU.end(), dp + o); o += LU.size();
    const size_t o_w = o; std::copy(at.w.begin(), at.w.end(), dp + o); o += at.w.size();
    std::copy(at.shift.begin(), at.shift.end(), reinterpret_cast<int*>(dp + o));
    if (hipMalloc(&h->tables, blob.size()) != hipSuccess) return bail(CHASM_ENOMEM, "hipMalloc(tables) failed");
    if (!by_transform && hipMalloc((void**)&h->D, D.size() * sizeof(double)) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(D) failed");
    if (by_transform && hipMalloc((void**)&h->tw, TW.size() * sizeof(fft::cd)) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(twiddles) failed");
    const size_t fb = (size_t)h->n * sizeof(double);
    if (hipMalloc((void**)&h->X, 2 * fb) != hipSuccess || hipMalloc((void**)&h->XA, 2 * fb) != hipSuccess ||
        (!by_transform &&
         (hipMalloc((void**)&h->Y, fb) != hipSuccess || hipMalloc((void**)&h->Z, fb) != hipSuccess)))
        return bail(CHASM_ENOMEM, "hipMalloc(state) failed");
    if (hipMemcpyAsync(h->tables, blob.data(), blob.size(), hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        (h->D && hipMemcpyAsync(h->D, D.data(), D.size() * sizeof(double), hipMemcpyHostToDevice, h->stream) !=
                     hipSuccess) ||
        (h->tw && hipMemcpyAsync(h->tw, TW.data(), TW.size() * sizeof(fft::cd), hipMemcpyHostToDevice, h->stream) !=
                      hipSuccess) ||
        hipStreamSynchronize(h->stream) != hipSuccess)
        return bail(CHASM_EDEVICE, "table upload failed");
    const double* tb = static_cast<const double*>(h->tables);
    HoArgs& a = h->args;
    a.N = d->nx;
    a.M = M;
    a.P = P;
    a.mlast = mlast;
    a.g = d->ghost;
    a.nk = d->nk;
    a.inflow = d->inflow;
    a.hx = d->hx;
    a.stencil = tb + o_st;
    a.lu = tb + o_lu;
    a.inv_l[0] = LM[M];
    a.ainv_l[0] = LM[2 * M + 1];
    a.inv_l[1] = LL[mlast];
    a.ainv_l[1] = LL[2 * mlast + 1];
    a.w = tb + o_w;
    a.shift = reinterpret_cast<const int*>(tb + o);
    *out = h;
    return CHASM_OK;
}

chasm_status chasm_ho2d_step(chasm_ho2d_t h, int32_t nsteps)
{
    if (!h) return hfail(CHASM_EINVAL, "handle is NULL");
    if (h->poisoned) return hfail(CHASM_ESTATE, "handle is poisoned by an earlier device failure");
    if (nsteps < 0) return hfail(CHASM_EINVAL, "nsteps must be >= 0");
    if (nsteps == 0) return CHASM_OK;
    const chasm_ho2d_desc& d = h->desc;
    const HoArgs& a = h->args;
    const long long n = h->n;
    const size_t fb = (size_t)n * sizeof(double);
    hipStream_t s = h->stream;
    double *F = h->X, *G = h->X + n, *FA = h->XA, *GA = h->XA + n;
    hipError_t e = hipSuccess;
    if (h->tw) {
        // Theta F; then per step: advect (F, Theta F); corrector fused with Theta (FA + tau
        // GA) and, but for the last step, with the next step's Theta F
        const DkArgs dp{d.nx, d.x_lo, d.hx, d.hk, d.omega, d.tau};
        const dim3 to((unsigned)((d.nx + 31) / 32), (unsigned)((d.nk + 31) / 32)), from(to.y, to.x);
        hipLaunchKernelGGL(k_ho_turn, to, dim3(256), 0, s, h->f, F, d.nk, d.nx);
        launch_dk(d.nk, DK_THETA, F, nullptr, nullptr, G, h->tw, dp, s);
        e = hipGetLastError();
        for (int it = 0; it < nsteps && e == hipSuccess; ++it) {
            launch_advect<true>(h->X, h->XA, a, s);
            launch_dk(d.nk, it + 1 < nsteps ? DK_STEP : DK_LAST, FA, GA, F, G, h->tw, dp, s);
            e = hipGetLastError();
        }
        if (e == hipSuccess) {
            hipLaunchKernelGGL(k_ho_turn, from, dim3(256), 0, s, F, h->f, d.nx, d.nk);
            e = hipGetLastError();
        }
    } else {
        const dim3 tgrid((unsigned)((d.nx + 31) / 32), (unsigned)((d.nk + 31) / 32));
        const unsigned cgrid = (unsigned)std::min<long long>((n + 255) / 256, 4096);
        e = hipMemcpyAsync(F, h->f, fb, hipMemcpyDeviceToDevice, s);
        for (int it = 0; it < nsteps && e == hipSuccess; ++it) {
            hipLaunchKernelGGL(k_ho_theta, tgrid, dim3(256), 0, s, h->D, F, G, d.nk, d.nx, d.x_lo, d.hx, d.omega);
            launch_advect<false>(h->X, h->XA, a, s);
            hipLaunchKernelGGL(k_ho_combine, dim3(cgrid), dim3(256), 0, s, h->Y, FA, GA, (const double*)nullptr, n, d.tau, 0);
            hipLaunchKernelGGL(k_ho_theta, tgrid, dim3(256), 0, s, h->D, h->Y, h->Z, d.nk, d.nx, d.x_lo, d.hx, d.omega);
            hipLaunchKernelGGL(k_ho_combine, dim3(cgrid), dim3(256), 0, s, F, FA, GA, h->Z, n, 0.5 * d.tau, 1);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipMemcpyAsync(h->f, F, fb, hipMemcpyDeviceToDevice, s);
    }
    if (e != hipSuccess) {
        h->poisoned = true;
        return hfail(CHASM_EDEVICE, std::string("ho2d step: ") + hipGetErrorString(e));
    }
    return CHASM_OK;
}

chasm_status chasm_ho2d_destroy(chasm_ho2d_t h)
{
    if (!h) return CHASM_OK;
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    for (void* p : {(void*)h->tables, (void*)h->D, (void*)h->tw, (void*)h->X, (void*)h->XA, (void*)h->Y, (void*)h->Z})
        if (p) (void)hipFree(p);
    delete h;
    return CHASM_OK;
}

}  // extern "C"
