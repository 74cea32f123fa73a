// chasm_marginals.hip -- the visualisation observables of Sec. 5: the reduced Wigner
// functions W_j(x_j, k_j) = integral of f over the other four variables, and the
// spatial marginal P(x1, x2) = integral of f over x3 and k, on the handle's field.
//
// Two passes, FP64, deterministic:
//   k_marg_item   one block per item (the x-cube of one (b, k)): the item's row of
//                 chasm_obs.hpp (column sums q over x3, plane sums G of 64-column
//                 groups), read once from HBM; each wave takes one 64-column group at
//                 a time, so every load of a wave is a contiguous run of x1;
//   k_marg_cols   P: 32 columns (x2, x1) to a block, 32 shares of the items, the sum of q;
//   k_marg_axes   per item, the row's contributions to the three W: a[x1] = sum of q over
//                 x2, b[x2] = sum of q over x1, c[x3] = sum of G over the groups, in place
//                 of values of the row that are no longer needed (axis_at);
//   k_marg_sum    one wave per W value, summing its items' contributions;
// all scaled by the cell volume of the integrated variables.
// Every sum runs in a fixed order.  One thread per output value, walking the item rows by
// itself, took 3.1 ms on 61^3 x 10^3 (59 MB of rows); the three take 12, 29 and 5 us.
// The x3 sweep that ends an observed step (CHASM_FLAG_OBSERVE) writes the same rows in
// its epilogue; the sums then complete the observables without reading the field.
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/chasm_advect.h"
#include "chasm_obs.hpp"

namespace chasm {

// A launch holds fewer than 2^32 threads: the kernels walk their units (items, column
// tiles, sums) with a grid of at most this many blocks.
constexpr long long kMargBlocks = 1LL << 20;

static dim3 marg_grid(long long units) { return dim3((unsigned)(units < kMargBlocks ? units : kMargBlocks)); }

template <typename T>
__global__ __launch_bounds__(256) void k_marg_item(const T* __restrict__ f, int n0, int n1, int n2, long long nitems,
                                                   double* __restrict__ part)
{
    const int plane = n0 * n1;
    const long long ngr = obs_groups(n0, n1);
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    for (long long item = blockIdx.x; item < nitems; item += gridDim.x) {
        const T* src = f + item * (long long)plane * n2;
        double* q = part + item * obs_row(n0, n1, n2);
        double* G = q + plane;
        for (long long g = wv; g < ngr; g += 4) {
            const long long c = 64 * g + ln;
            const bool in = c < plane;
            double acc = 0.0;
            for (int z = 0; z < n2; ++z) {
                const double x = in ? (double)src[(long long)z * plane + c] : 0.0;
                acc += x;
                const double gs = obs_wave_sum(x);
                if (ln == 0) G[g * n2 + z] = gs;
            }
            if (in) q[c] = acc;
        }
    }
}

struct MargArgs {
    int nx[3], nk[3], nbatch;
    double s[4];                 // cell volumes of the integrated variables: W1, W2, W3, P
};

// out layout per batch member b: W1[k1][x1] | W2[k2][x2] | W3[k3][x3] | P[x2][x1].
__host__ __device__ __forceinline__ long long marg_w(const MargArgs& a)
{
    return (long long)a.nx[0] * a.nk[0] + (long long)a.nx[1] * a.nk[1] + (long long)a.nx[2] * a.nk[2];
}

__global__ __launch_bounds__(1024) void k_marg_cols(const double* __restrict__ part, MargArgs a, double* __restrict__ out)
{
    __shared__ double red[32][33];
    const long long plane = (long long)a.nx[0] * a.nx[1], nkp = (long long)a.nk[0] * a.nk[1] * a.nk[2];
    const long long tiles = (plane + 31) / 32, row = obs_row(a.nx[0], a.nx[1], a.nx[2]);
    const int cl = threadIdx.x % 32, sh = threadIdx.x / 32;
    for (long long tile = blockIdx.x; tile < tiles * a.nbatch; tile += gridDim.x) {
        const long long b = tile / tiles, c = tile % tiles * 32 + cl;
        double t = 0.0;
        if (c < plane) {
            const double* q = part + b * nkp * row + c;
#pragma unroll 8
            for (long long i = sh; i < nkp; i += 32) t += q[i * row];
        }
        red[sh][cl] = t;
        __syncthreads();
        if (sh == 0 && c < plane) {
            double p = 0.0;
            for (int u = 0; u < 32; ++u) p += red[u][cl];
            out[b * (marg_w(a) + plane) + marg_w(a) + c] = p * a.s[3];
        }
        __syncthreads();
    }
}

// Where k_marg_axes leaves node j of axis d in an item's row: a over row 0 of q, b[y] over
// the first value of row y (b[0] over the second of row 1), c over group 0 of G.
__device__ __forceinline__ long long axis_at(const MargArgs& a, int d, int j)
{
    const long long N0 = a.nx[0];
    return d == 0 ? j : d == 1 ? (j ? j * N0 : N0 + 1) : N0 * a.nx[1] + j;
}

__global__ __launch_bounds__(256) void k_marg_axes(double* __restrict__ part, MargArgs a)
{
    __shared__ double red[4][64];
    const int N0 = a.nx[0], N1 = a.nx[1], N2 = a.nx[2];
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    auto across = [&](const double* q, int y) {      // sum of row y, by a wave
        double t = 0.0;
        for (int x = ln; x < N0; x += 64) t += q[(long long)y * N0 + x];
        return obs_wave_sum(t);
    };
    // sums down the columns of a rows x cols matrix into its row 0, 64 columns at a time:
    // wave w takes the rows w, w + 4, ...; the four partial sums are added in wave order
    auto down = [&](double* m, long long rows, int cols) {
        for (int c0 = 0; c0 < cols; c0 += 64) {
            const int c = c0 + ln;
            double t = 0.0;
            if (c < cols)
                for (long long r = wv; r < rows; r += 4) t += m[r * cols + c];
            red[wv][ln] = t;
            __syncthreads();
            if (wv == 0 && c < cols) m[c] = (red[0][ln] + red[1][ln]) + (red[2][ln] + red[3][ln]);
            __syncthreads();
        }
    };
    const long long nitems = (long long)a.nk[0] * a.nk[1] * a.nk[2] * a.nbatch;
    for (long long item = blockIdx.x; item < nitems; item += gridDim.x) {
        double* q = part + item * obs_row(N0, N1, N2);
        const double b0 = across(q, 0);              // before row 0 is overwritten
        __syncthreads();
        down(q, N1, N0);
        down(q + (long long)N0 * N1, obs_groups(N0, N1), N2);
        for (int y = wv; y < N1; y += 4) {
            if (y == 0) continue;
            const double t = across(q, y);           // row y is read and written by this wave alone
            if (ln == 0) {
                q[axis_at(a, 1, y)] = t;
                if (y == 1) q[axis_at(a, 1, 0)] = b0;
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_marg_sum(const double* __restrict__ part, MargArgs a, double* __restrict__ out)
{
    const long long plane = (long long)a.nx[0] * a.nx[1], nkp = (long long)a.nk[0] * a.nk[1] * a.nk[2];
    const long long nw = marg_w(a), row = obs_row(a.nx[0], a.nx[1], a.nx[2]);
    const int ln = threadIdx.x & 63;
    for (long long id = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); id < nw * a.nbatch; id += (long long)gridDim.x * 4) {
        const long long b = id / nw;
        long long r = id % nw;
        // axis d, its node j and k index kd; the items of kd
        int d = 0;
        while (d < 2 && r >= (long long)a.nx[d] * a.nk[d]) r -= (long long)a.nx[d] * a.nk[d++];
        const long long kd = r / a.nx[d];
        const long long inner = d == 0 ? 1 : d == 1 ? a.nk[0] : (long long)a.nk[0] * a.nk[1];   // stride of k_d
        const long long rest = nkp / a.nk[d];
        const double* v = part + b * nkp * row + axis_at(a, d, (int)(r % a.nx[d]));
        double t = 0.0;
        for (long long u = ln; u < rest; u += 64) t += v[((u / inner) * inner * a.nk[d] + kd * inner + u % inner) * row];
        t = obs_wave_sum(t);
        if (ln == 0) out[b * (nw + plane) + id % nw] = t * a.s[d];
    }
}

// Doubles of an item row.
long long marginal_row(const int nx[3]) { return obs_row(nx[0], nx[1], nx[2]); }

// All passes on stream st: part holds the item rows (marginal_row(nx) doubles each), which
// the sums use up, out nbatch * (nx1 nk1 + nx2 nk2 + nx3 nk3 + nx1 nx2) doubles.  f
// nullptr: the item rows are already in part (written by an observing x3 sweep).
hipError_t launch_marginals(int dtype, const int nx[3], const int nk[3], int nbatch, const double hx[3],
                            const double hk[3], const void* f, double* part, double* out, hipStream_t st)
{
    const long long nitems = (long long)nk[0] * nk[1] * nk[2] * nbatch;
    if (f) {
        if (dtype == CHASM_F64)
            hipLaunchKernelGGL((k_marg_item<double>), marg_grid(nitems), dim3(256), 0, st,
                               static_cast<const double*>(f), nx[0], nx[1], nx[2], nitems, part);
        else
            hipLaunchKernelGGL((k_marg_item<float>), marg_grid(nitems), dim3(256), 0, st,
                               static_cast<const float*>(f), nx[0], nx[1], nx[2], nitems, part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    MargArgs a{};
    a.nbatch = nbatch;
    for (int d = 0; d < 3; ++d) {
        a.nx[d] = nx[d];
        a.nk[d] = nk[d];
    }
    const double v[3] = {hx[0] * hk[0], hx[1] * hk[1], hx[2] * hk[2]};
    a.s[0] = v[1] * v[2];
    a.s[1] = v[0] * v[2];
    a.s[2] = v[0] * v[1];
    a.s[3] = hx[2] * hk[0] * hk[1] * hk[2];
    const long long plane = (long long)nx[0] * nx[1];
    hipLaunchKernelGGL(k_marg_cols, marg_grid((plane + 31) / 32 * nbatch), dim3(1024), 0, st, part, a, out);
    hipLaunchKernelGGL(k_marg_axes, marg_grid(nitems), dim3(256), 0, st, part, a);
    hipLaunchKernelGGL(k_marg_sum, marg_grid((marg_w(a) * nbatch + 3) / 4), dim3(256), 0, st, part, a, out);
    return hipGetLastError();
}

}  // namespace chasm
