// chasm_marginals.hip -- the visualisation observables of Sec. 5: the reduced Wigner
// functions W_j(x_j, k_j) = integral of f over the other four variables, and the
// spatial marginal P(x1, x2) = integral of f over x3 and k, on the handle's field.
//
// Two passes, FP64, deterministic:
//   k_marg_item   one block per item (the x-cube of one (b, k)): the item's row of
//                 chasm_obs.hpp (column sums q over x3, plane sums G of 64-column
//                 groups), read once from HBM; each wave takes one 64-column group at
//                 a time, so every load of a wave is a contiguous run of x1;
//   k_marg_axes   per item, the row's contributions to the three W: a[x1] = sum of q over
//                 x2, b[x2] = sum of q over x1, c[x3] = sum of G over the groups;
//   k_marg_cols   P: one thread per column (x2, x1) and chunk of items, the sum of q;
//   k_marg_sum    one wave per W value, summing its items' contributions, and one thread
//                 per P value, summing the chunks; scales by the cell volume of the
//                 integrated variables.
// Every sum runs in a fixed order.  One thread per output value, walking the item rows by
// itself, took 3.1 ms on 61^3 x 10^3 (59 MB of rows); k_marg_axes 32 us, k_marg_cols 7 and
// k_marg_sum 18 take its place.
// The x3 sweep that ends an observed step (CHASM_FLAG_OBSERVE) writes the same rows in
// its epilogue; the sums then complete the observables without reading the field.
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/chasm_advect.h"
#include "chasm_obs.hpp"

namespace chasm {

template <typename T>
__global__ __launch_bounds__(256) void k_marg_item(const T* __restrict__ f, int n0, int n1, int n2,
                                                   double* __restrict__ part)
{
    const int plane = n0 * n1;
    const long long ngr = obs_groups(n0, n1);
    const long long item = blockIdx.x;
    const T* src = f + item * (long long)plane * n2;
    double* q = part + item * obs_row(n0, n1, n2);
    double* G = q + plane;
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
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

struct MargArgs {
    int nx[3], nk[3], nbatch;
    double s[4];                 // cell volumes of the integrated variables: W1, W2, W3, P
    int chunks;                  // of the items of a batch member, for P
};

// Doubles of the second stage's workspace: per item a | b | c, then per chunk of a batch
// member's items the partial P.
static long long marg_axes(const int nx[3]) { return (long long)nx[0] + nx[1] + nx[2]; }

// Chunks of a batch member's nkp items: enough threads for the chip, at least 16 items each.
static int marg_chunks(const int nx[3], long long nkp)
{
    const long long want = (256LL * 2048) / ((long long)nx[0] * nx[1]) + 1;
    const long long most = (nkp + 15) / 16;
    return (int)(want < most ? want : most);
}

__global__ __launch_bounds__(256) void k_marg_axes(const double* __restrict__ part, MargArgs a, double* __restrict__ axes)
{
    __shared__ double red[4][64];
    const int N0 = a.nx[0], N1 = a.nx[1], N2 = a.nx[2];
    const long long item = blockIdx.x;
    const double* q = part + item * obs_row(N0, N1, N2);
    const double* G = q + (long long)N0 * N1;
    double* out = axes + item * (N0 + N1 + N2);
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
    // sums down the columns of a rows x cols matrix, 64 columns at a time: wave w takes the
    // rows w, w + 4, ...; the four partial sums are added in wave order
    auto down = [&](const double* m, long long rows, int cols, double* dst) {
        for (int c0 = 0; c0 < cols; c0 += 64) {
            const int c = c0 + ln;
            double t = 0.0;
            if (c < cols)
                for (long long r = wv; r < rows; r += 4) t += m[r * cols + c];
            red[wv][ln] = t;
            __syncthreads();
            if (wv == 0 && c < cols) dst[c] = (red[0][ln] + red[1][ln]) + (red[2][ln] + red[3][ln]);
            __syncthreads();
        }
    };
    down(q, N1, N0, out);
    down(G, obs_groups(N0, N1), N2, out + N0 + N1);
    for (int y = wv; y < N1; y += 4) {               // a wave per row
        double t = 0.0;
        for (int x = ln; x < N0; x += 64) t += q[(long long)y * N0 + x];
        t = obs_wave_sum(t);
        if (ln == 0) out[N0 + y] = t;
    }
}

__global__ __launch_bounds__(256) void k_marg_cols(const double* __restrict__ part, MargArgs a, double* __restrict__ cols)
{
    const long long plane = (long long)a.nx[0] * a.nx[1], nkp = (long long)a.nk[0] * a.nk[1] * a.nk[2];
    const unsigned tiles = (unsigned)((plane + 255) / 256), u = blockIdx.x / tiles;
    const long long c = (long long)(blockIdx.x % tiles) * 256 + threadIdx.x;
    if (c >= plane) return;
    const long long ch = u % a.chunks, b = u / a.chunks;
    const long long per = (nkp + a.chunks - 1) / a.chunks, i0 = ch * per, i1 = i0 + per < nkp ? i0 + per : nkp;
    const long long row = obs_row(a.nx[0], a.nx[1], a.nx[2]);
    const double* q = part + b * nkp * row + c;
    double t = 0.0;
#pragma unroll 8
    for (long long i = i0; i < i1; ++i) t += q[i * row];
    cols[((long long)b * a.chunks + ch) * plane + c] = t;
}

// out layout per batch member b: W1[k1][x1] | W2[k2][x2] | W3[k3][x3] | P[x2][x1].
__global__ __launch_bounds__(256) void k_marg_sum(const double* __restrict__ axes, const double* __restrict__ cols,
                                                  MargArgs a, double* __restrict__ out)
{
    const int N0 = a.nx[0], N1 = a.nx[1], N2 = a.nx[2], n1 = a.nk[0], n2 = a.nk[1], n3 = a.nk[2];
    const long long plane = (long long)N0 * N1, nkp = (long long)n1 * n2 * n3;
    const long long nw = (long long)N0 * n1 + (long long)N1 * n2 + (long long)N2 * n3, per_b = nw + plane;
    const long long wblocks = (nw * a.nbatch + 3) / 4;
    const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63, A = N0 + N1 + N2;
    if (blockIdx.x < wblocks) {                      // a wave per W value
        const long long id = (long long)blockIdx.x * 4 + wv;
        if (id >= nw * a.nbatch) return;
        const int b = (int)(id / nw);
        long long r = id % nw;
        const double* base = axes + b * nkp * A;
        // axis d, its node j and k index kd; the items of kd: i = lo + hi * stride
        int d = 0;
        const int N[3] = {N0, N1, N2}, n[3] = {n1, n2, n3};
        while (d < 2 && r >= (long long)N[d] * n[d]) r -= (long long)N[d] * n[d++];
        const int kd = (int)(r / N[d]), j = (int)(r % N[d]);
        const long long inner = d == 0 ? 1 : d == 1 ? n1 : (long long)n1 * n2;   // stride of k_d
        const long long rest = nkp / n[d];
        const double* v = base + (d == 0 ? 0 : d == 1 ? N0 : N0 + N1) + j;
        double t = 0.0;
        for (long long u = ln; u < rest; u += 64) {
            const long long i = (u / inner) * inner * n[d] + kd * inner + u % inner;
            t += v[i * A];
        }
        t = obs_wave_sum(t);
        if (ln == 0) out[b * per_b + id % nw] = t * a.s[d];
    } else {                                         // a thread per P value
        const long long id = ((long long)blockIdx.x - wblocks) * 256 + threadIdx.x;
        if (id >= plane * a.nbatch) return;
        const long long b = id / plane, c = id % plane;
        double t = 0.0;
        for (int ch = 0; ch < a.chunks; ++ch) t += cols[(b * a.chunks + ch) * plane + c];
        out[b * per_b + nw + c] = t * a.s[3];
    }
}

// Doubles of the workspace of a field's marginals: the item rows (chasm_obs.hpp), then the
// second stage's sums.
long long marginal_workspace(const int nx[3], const int nk[3], int nbatch)
{
    const long long nkp = (long long)nk[0] * nk[1] * nk[2];
    return nkp * nbatch * (obs_row(nx[0], nx[1], nx[2]) + marg_axes(nx)) +
           (long long)marg_chunks(nx, nkp) * nbatch * nx[0] * nx[1];
}

// All passes on stream st: part holds marginal_workspace(nx, nk, nbatch) doubles, out
// nbatch * (nx1 nk1 + nx2 nk2 + nx3 nk3 + nx1 nx2) doubles.  f nullptr: the item rows
// are already in part (written by an observing x3 sweep); only the sums run.
hipError_t launch_marginals(int dtype, const int nx[3], const int nk[3], int nbatch, const double hx[3],
                            const double hk[3], const void* f, double* part, double* out, hipStream_t st)
{
    const long long nitems = (long long)nk[0] * nk[1] * nk[2] * nbatch;
    if (f) {
        if (dtype == CHASM_F64)
            hipLaunchKernelGGL((k_marg_item<double>), dim3((unsigned)nitems), dim3(256), 0, st,
                               static_cast<const double*>(f), nx[0], nx[1], nx[2], part);
        else
            hipLaunchKernelGGL((k_marg_item<float>), dim3((unsigned)nitems), dim3(256), 0, st,
                               static_cast<const float*>(f), nx[0], nx[1], nx[2], part);
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
    const long long nkp = (long long)nk[0] * nk[1] * nk[2], plane = (long long)nx[0] * nx[1];
    const long long nw = (long long)nx[0] * nk[0] + (long long)nx[1] * nk[1] + (long long)nx[2] * nk[2];
    a.chunks = marg_chunks(nx, nkp);
    double* const axes = part + nitems * obs_row(nx[0], nx[1], nx[2]);
    double* const cols = axes + nitems * marg_axes(nx);
    hipLaunchKernelGGL(k_marg_axes, dim3((unsigned)nitems), dim3(256), 0, st, part, a, axes);
    hipLaunchKernelGGL(k_marg_cols, dim3((unsigned)((plane + 255) / 256 * a.chunks * nbatch)), dim3(256), 0, st, part, a,
                       cols);
    hipLaunchKernelGGL(k_marg_sum, dim3((unsigned)((nw * nbatch + 3) / 4 + (plane * nbatch + 255) / 256)), dim3(256), 0, st,
                       axes, cols, a, out);
    return hipGetLastError();
}

}  // namespace chasm
