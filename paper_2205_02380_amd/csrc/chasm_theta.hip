// chasm_theta.hip -- C ABI of the truncated-kernel evaluation of Theta_V (Sec. 4):
// descriptor validation, the FP64 tensor T of eq. 4.9 on the host, kernel selection, and
// the apply sequence (transpose to x-major, kernel tables and convolutions over ranges of
// x-points, transpose back).  See include/chasm_theta.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <complex>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/chasm_theta.h"
#include "chasm_theta_launch.hpp"

namespace chasm {

void set_last_error(const std::string& msg);

// ---------------------------------------------------------------------------
// Sine integral Si(x) = int_0^x sin(t)/t dt.  |x| <= 4: the Maclaurin series
// sum_n (-1)^n x^{2n+1} / ((2n+1) (2n+1)!).  Beyond: Si(x) = pi/2 + Im E1(i x)
// (E1(i x) = -Ci(x) + i (Si(x) - pi/2)), with E1 from its continued fraction
// e^{z} E1(z) = 1/(z+1 - 1/(z+3 - 4/(z+5 - 9/(z+7 - ...)))) evaluated by the modified
// Lentz method.
static double sine_integral(double x)
{
    const double ax = std::fabs(x);
    double r;
    if (ax <= 4.0) {
        double p = ax, sum = ax;
        for (int n = 1; n < 60; ++n) {
            p *= -ax * ax / ((2.0 * n) * (2.0 * n + 1.0));
            const double t = p / (2.0 * n + 1.0);
            sum += t;
            if (std::fabs(t) < 1e-18 * std::fabs(sum)) break;
        }
        r = sum;
    } else {
        const std::complex<double> z(0.0, ax);
        const double tiny = 1e-300;
        std::complex<double> b = z + 1.0, c = 1.0 / tiny, d = 1.0 / b, h = d;
        for (int i = 1; i < 10000; ++i) {
            const double an = -(double)i * (double)i;
            b += 2.0;
            d = 1.0 / (an * d + b);
            c = b + an / c;
            const std::complex<double> del = c * d;
            h *= del;
            if (std::abs(del - 1.0) < 1e-16) break;
        }
        r = M_PI / 2 + (h * std::exp(-z)).imag();
    }
    return x < 0 ? -r : r;
}

// Fourier transform of |k|^-2 truncated at |k| <= D, at |xi| = q (Sec. 4.1).
static double uhat_truncated(double q, double D)
{
    return q > 0 ? 4.0 * M_PI * sine_integral(q * D) / q : 4.0 * M_PI * D;
}

// cos(2 pi a / m) with a reduced modulo m first.
static double cos_turn(long long a, long long m)
{
    a %= m;
    if (a < 0) a += m;
    return std::cos(2.0 * M_PI * (double)a / (double)m);
}

// T_p of eq. 4.9 for p_d in [0, nk_d): the real sum (1/M^3) sum_n Uhat_D(xi_n)
// prod_d cos(2 pi p_d n_d / M_d) over the dual set n_d in [-M_d/2, M_d/2), M_d = 3 nk_d,
// xi_{n,d} = 2 pi n_d / (M_d hk_d) (eq. 4.10), in three separable passes.  The odd
// parts cancel between n_d and -n_d, and the unpaired n_d = -M_d/2 has a zero sine.
// Output [p3][p2][p1]; T is even in every p_d.
static void tensor_positive(const int nk[3], const double hk[3], std::vector<double>& T)
{
    const int M[3] = {3 * nk[0], 3 * nk[1], 3 * nk[2]};
    double D2 = 0.0;
    for (int d = 0; d < 3; ++d) D2 += (nk[d] * hk[d]) * (nk[d] * hk[d]);
    const double D = std::sqrt(D2);
    std::vector<double> xi[3];
    for (int d = 0; d < 3; ++d) {
        xi[d].resize(M[d]);
        for (int i = 0; i < M[d]; ++i) xi[d][i] = 2.0 * M_PI * (i - M[d] / 2) / (M[d] * hk[d]);
    }
    std::vector<double> cs[3];   // cs[d][p * M + i] = cos(2 pi p n_i / M)
    for (int d = 0; d < 3; ++d) {
        cs[d].resize((size_t)nk[d] * M[d]);
        for (int p = 0; p < nk[d]; ++p)
            for (int i = 0; i < M[d]; ++i) cs[d][(size_t)p * M[d] + i] = cos_turn((long long)p * (i - M[d] / 2), M[d]);
    }
    // pass 1 over n1: A1[n3][n2][p1]
    std::vector<double> A1((size_t)M[2] * M[1] * nk[0]);
    std::vector<double> U(M[0]);
    for (int i3 = 0; i3 < M[2]; ++i3)
        for (int i2 = 0; i2 < M[1]; ++i2) {
            for (int i1 = 0; i1 < M[0]; ++i1)
                U[i1] = uhat_truncated(std::sqrt(xi[0][i1] * xi[0][i1] + xi[1][i2] * xi[1][i2] + xi[2][i3] * xi[2][i3]), D);
            for (int p1 = 0; p1 < nk[0]; ++p1) {
                double s = 0.0;
                for (int i1 = 0; i1 < M[0]; ++i1) s += U[i1] * cs[0][(size_t)p1 * M[0] + i1];
                A1[((size_t)i3 * M[1] + i2) * nk[0] + p1] = s;
            }
        }
    // pass 2 over n2: A2[n3][p2][p1]
    std::vector<double> A2((size_t)M[2] * nk[1] * nk[0]);
    for (int i3 = 0; i3 < M[2]; ++i3)
        for (int p2 = 0; p2 < nk[1]; ++p2)
            for (int p1 = 0; p1 < nk[0]; ++p1) {
                double s = 0.0;
                for (int i2 = 0; i2 < M[1]; ++i2)
                    s += A1[((size_t)i3 * M[1] + i2) * nk[0] + p1] * cs[1][(size_t)p2 * M[1] + i2];
                A2[((size_t)i3 * nk[1] + p2) * nk[0] + p1] = s;
            }
    // pass 3 over n3, with the 1/M^3 of the inverse DFT
    const double scale = 1.0 / ((double)M[0] * M[1] * M[2]);
    T.assign((size_t)nk[2] * nk[1] * nk[0], 0.0);
    for (int p3 = 0; p3 < nk[2]; ++p3)
        for (int p2 = 0; p2 < nk[1]; ++p2)
            for (int p1 = 0; p1 < nk[0]; ++p1) {
                double s = 0.0;
                for (int i3 = 0; i3 < M[2]; ++i3)
                    s += A2[((size_t)i3 * nk[1] + p2) * nk[0] + p1] * cs[2][(size_t)p3 * M[2] + i3];
                T[((size_t)p3 * nk[1] + p2) * nk[0] + p1] = s * scale;
            }
}

// The kernels of (dtype, nk), or nullptr.
static const ThetaKernels* find_theta(int dtype, int nk)
{
    const ThetaKernels* k = nk == 8 ? theta_kernels_8() : nk == 16 ? theta_kernels_16() : nk == 32 ? theta_kernels_32()
                            : nk == 64 ? theta_kernels_64() : nullptr;
    return k ? &k[dtype == CHASM_F64 ? 1 : 0] : nullptr;
}

// How a handle goes through its x-points (order t, chasm_theta.hpp): the tables of at most
// np pairs and, staged, an intermediate W of X x-points at a time.
//   Tables: 4 nk^3 doubles per pair and nucleus, 128 MiB at most (two pairs at least).  If
//   that holds all pairs they are made once, at create; else for each range of each call,
//   which costs a pair as much as the Toeplitz products of one of its nx3 nbatch x-points.
//   U, 2 nk^3 doubles per x1 node and nucleus, likewise.
//   W: 192 MiB at most.  18^3 x 32^3 with two nuclei, whose ranges have 42 MiB of tables, takes
//   5.33 ms, against 5.44 at 256 MiB, 5.55 at 128 and 6.45 at 64 (launch gaps and half-empty
//   rounds): W and the tables then stay in the 256 MB memory-side cache between the stages.
//   With three or four x-points to a pair the tables of a range are up to their own bound
//   and the two exceed it.
struct ThetaPlan {
    bool big, resident, u_resident;
    int np;
    long long X;
    size_t tab, U, W;                   // bytes
};

static bool use_big(const chasm_theta_desc* d, const ThetaKernels* ks);

static ThetaPlan theta_plan(const chasm_theta_desc* d, const ThetaKernels* ks)
{
    ThetaPlan p{};
    p.big = use_big(d, ks);
    const long long cube = (long long)d->nk[0] * d->nk[1] * d->nk[2];
    const long long pairs = (long long)d->nx[0] * d->nx[1], m = (long long)d->nx[2] * d->nbatch;
    const long long per_pair = 4 * cube * 8 * d->nnuc, per_node = 2 * cube * 8 * d->nnuc;
    long long most = (128LL << 20) / per_pair;
    if (most < 2) most = 2;
    p.resident = most >= pairs;
    const long long ranges = (pairs + most - 1) / most;
    p.X = (pairs + ranges - 1) / ranges * m;            // ranges of equal size
    if (p.big) {
        const long long x = (192LL << 20) / (16 * cube);
        if (x < p.X) p.X = x < 1 ? 1 : x;
        if (p.X >= m) p.X -= p.X % m;                   // whole pairs
    }
    long long np = p.X >= m ? p.X / m : 2;
    if (p.resident || np > pairs) np = pairs;
    p.np = (int)np;
    long long nodes = np / d->nx[1] + 2;                // x1 nodes of a range
    p.u_resident = nodes >= d->nx[0] || per_node * d->nx[0] <= 128LL << 20;
    if (p.u_resident) nodes = d->nx[0];
    p.tab = (size_t)(np * per_pair);
    p.U = (size_t)(nodes * per_node);
    p.W = p.big ? (size_t)(p.X * cube * 16) : 0;
    return p;
}

static bool use_big(const chasm_theta_desc* d, const ThetaKernels* ks)
{
    return !ks->theta || (d->flags & CHASM_THETA_FLAG_STAGED);
}

}  // namespace chasm

using namespace chasm;

struct chasm_theta_s {
    chasm_theta_desc desc;
    hipStream_t stream = nullptr;
    const ThetaKernels* ks = nullptr;
    ThetaPlan plan{};
    double* T = nullptr;                // tensor, [q1][q2][q3]
    fft::cd* et = nullptr;              // factors of the grid's nodes (k_theta_mod)
    double *tab = nullptr, *U = nullptr;   // kernel tables (chasm_theta_table.hpp) and their first sum
    void* ws = nullptr;
    fft::cd* W = nullptr;               // complex intermediate of the staged form
    ThetaArgs args{};
    long long npts = 0, nkp = 0;
    bool poisoned = false;
};

static chasm_status tfail(chasm_status st, const std::string& msg)
{
    set_last_error(msg);
    return st;
}

static chasm_status validate(const chasm_theta_desc* d, const ThetaKernels** ks)
{
    if (!d) return tfail(CHASM_EINVAL, "descriptor is NULL");
    for (int a = 0; a < 3; ++a) {
        if (d->nx[a] < 1 || d->nk[a] < 2) return tfail(CHASM_EINVAL, "nx must be >= 1 and nk >= 2 on every axis");
        if (!(d->x_hi[a] > d->x_lo[a]) || !(d->k_hi[a] > d->k_lo[a]) || !std::isfinite(d->x_lo[a]) ||
            !std::isfinite(d->x_hi[a]) || !std::isfinite(d->k_lo[a]) || !std::isfinite(d->k_hi[a]))
            return tfail(CHASM_EINVAL, "every axis needs finite bounds with hi > lo");
        if (d->nk[a] % 2) return tfail(CHASM_EINVAL, "nk must be even (the dual index set of eq. 4.10)");
    }
    if (d->nnuc < 1 || d->nnuc > CHASM_THETA_MAX_NUCLEI) return tfail(CHASM_EINVAL, "nnuc must be in 1..4");
    for (int i = 0; i < d->nnuc; ++i) {
        if (!std::isfinite(d->z_nuc[i])) return tfail(CHASM_EINVAL, "nucleus charge is not finite");
        for (int a = 0; a < 3; ++a)
            if (!std::isfinite(d->x_nuc[i][a])) return tfail(CHASM_EINVAL, "nucleus position is not finite");
    }
    if (d->dtype != CHASM_F32 && d->dtype != CHASM_F64) return tfail(CHASM_EINVAL, "dtype must be CHASM_F32 or CHASM_F64");
    if (d->nbatch < 1) return tfail(CHASM_EINVAL, "nbatch must be >= 1");
    const long long pts = (long long)d->nx[0] * d->nx[1] * d->nx[2] * d->nk[0] * d->nk[1] * d->nk[2];
    if (pts <= 0 || pts > (1LL << 40) / d->nbatch) return tfail(CHASM_EINVAL, "grid too large");
    if (d->flags & ~(uint32_t)CHASM_THETA_FLAG_STAGED) return tfail(CHASM_EINVAL, "unknown flags");
    if (d->nk[0] != d->nk[1] || d->nk[1] != d->nk[2])
        return tfail(CHASM_EUNSUPPORTED, "kernels are built for equal nk on the three axes");
    const ThetaKernels* k = find_theta(d->dtype, d->nk[0]);
    if (!k) return tfail(CHASM_EUNSUPPORTED, "no kernel for this nk (built: 8, 16, 32, 64)");
    if ((d->flags & CHASM_THETA_FLAG_STAGED) && !k->big)
        return tfail(CHASM_EUNSUPPORTED, "the staged form is built for nk 16, 32, 64");
    if (ks) *ks = k;
    return CHASM_OK;
}

static void desc_hk(const chasm_theta_desc* d, int nk[3], double hk[3])
{
    for (int a = 0; a < 3; ++a) {
        nk[a] = d->nk[a];
        hk[a] = (d->k_hi[a] - d->k_lo[a]) / d->nk[a];
    }
}

static hipError_t make_tables(chasm_theta_t h, const ThetaRange& r)
{
    int i1_0 = 0;
    if (!h->plan.u_resident) {
        const int nx2 = h->desc.nx[1];
        i1_0 = r.p0 / nx2;
        const hipError_t e = h->ks->node(h->U, h->T, h->et, h->args, i1_0, (r.p0 + r.np - 1) / nx2 - i1_0 + 1, h->stream);
        if (e != hipSuccess) return e;
    }
    return h->ks->table(h->tab, h->U, h->et, h->args, r, i1_0, h->stream);
}

// The convolutions of all x-points on the x-major copy, range by range.
static hipError_t convolve(chasm_theta_t h)
{
    const ThetaPlan& p = h->plan;
    const long long m = (long long)h->desc.nx[2] * h->desc.nbatch, total = h->npts * h->desc.nbatch;
    ThetaRange r{0, 0, 0, 0};
    if (p.resident) r.np = p.np;
    for (; r.t0 < total; r.t0 += p.X) {
        r.n = total - r.t0 < p.X ? total - r.t0 : p.X;
        hipError_t e = hipSuccess;
        if (!p.resident) {
            const int p0 = (int)(r.t0 / m), np = (int)((r.t0 + r.n - 1) / m) - p0 + 1;
            const bool made = p0 == r.p0 && np == r.np;   // ranges within one pair
            r.p0 = p0;
            r.np = np;
            if (!made) e = make_tables(h, r);
        }
        if (e == hipSuccess)
            e = p.big ? h->ks->big(h->ws, h->tab, h->et, h->args, r, h->W, h->stream)
                      : h->ks->theta(h->ws, h->tab, h->et, h->args, r, h->stream);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// x-major copy (mode_in), the convolutions on it, and back (mode_out); see TransposeMode.
static chasm_status run_theta(chasm_theta_t h, int mode_in, const void* f, const void* g_in, double c_in, int mode_out,
                              void* out, const void* g_out, double c_out)
{
    const int nb = h->desc.nbatch;
    hipError_t e = h->ks->transpose(mode_in, f, g_in, h->ws, h->nkp, h->npts, nb, c_in, h->stream);
    if (e == hipSuccess) e = convolve(h);
    if (e == hipSuccess) e = h->ks->transpose(mode_out, h->ws, g_out, out, h->npts, h->nkp, nb, c_out, h->stream);
    if (e != hipSuccess) {
        h->poisoned = true;
        return tfail(CHASM_EDEVICE, std::string("theta launch: ") + hipGetErrorString(e));
    }
    return CHASM_OK;
}

namespace chasm {
// The predictor and corrector of an LPC1 step: f = f + tau/2 (g + Theta[f + tau g]).
chasm_status theta_lpc1(chasm_theta_t h, void* f, const void* g, double tau)
{
    if (h->poisoned) return tfail(CHASM_ESTATE, "handle is poisoned by an earlier device failure");
    return run_theta(h, TR_PREDICT, f, g, tau, TR_CORRECT, f, g, 0.5 * tau);
}
}  // namespace chasm

extern "C" {

chasm_status chasm_theta_workspace_bytes(const chasm_theta_desc* desc, size_t* bytes)
{
    const ThetaKernels* ks = nullptr;
    chasm_status st = validate(desc, &ks);
    if (st != CHASM_OK) return st;
    if (!bytes) return tfail(CHASM_EINVAL, "bytes is NULL");
    const size_t es = desc->dtype == CHASM_F64 ? 8 : 4;
    const size_t pts = (size_t)desc->nx[0] * desc->nx[1] * desc->nx[2] * desc->nk[0] * desc->nk[1] * desc->nk[2];
    const ThetaPlan p = theta_plan(desc, ks);
    const size_t nrow = (size_t)desc->nx[0] + desc->nx[1] + desc->nx[2], cube = (size_t)desc->nk[0] * desc->nk[1] * desc->nk[2];
    *bytes = pts * desc->nbatch * es + cube * sizeof(double) + (4 + (size_t)desc->nnuc * nrow) * desc->nk[0] * sizeof(fft::cd) +
             p.tab + p.U + p.W + 6 * 256;
    return CHASM_OK;
}

chasm_status chasm_theta_tensor(const chasm_theta_desc* desc, double* t_host)
{
    chasm_status st = validate(desc, nullptr);
    if (st != CHASM_OK && st != CHASM_EUNSUPPORTED) return st;
    if (!t_host) return tfail(CHASM_EINVAL, "t_host is NULL");
    int nk[3];
    double hk[3];
    desc_hk(desc, nk, hk);
    std::vector<double> T;
    tensor_positive(nk, hk, T);
    const int w1 = 2 * nk[0] - 1, w2 = 2 * nk[1] - 1, w3 = 2 * nk[2] - 1;
    for (int q3 = 0; q3 < w3; ++q3)
        for (int q2 = 0; q2 < w2; ++q2)
            for (int q1 = 0; q1 < w1; ++q1) {
                const int p3 = std::abs(q3 - (nk[2] - 1)), p2 = std::abs(q2 - (nk[1] - 1)), p1 = std::abs(q1 - (nk[0] - 1));
                t_host[((size_t)q3 * w2 + q2) * w1 + q1] = T[((size_t)p3 * nk[1] + p2) * nk[0] + p1];
            }
    return CHASM_OK;
}

chasm_status chasm_theta_create(const chasm_theta_desc* desc, void* hip_stream, chasm_theta_t* out)
{
    if (!out) return tfail(CHASM_EINVAL, "out is NULL");
    *out = nullptr;
    const ThetaKernels* ks = nullptr;
    chasm_status st = validate(desc, &ks);
    if (st != CHASM_OK) return st;

    int nk[3];
    double hk[3];
    desc_hk(desc, nk, hk);
    std::vector<double> T, TQ;
    tensor_positive(nk, hk, T);
    TQ.resize(T.size());
    for (int q3 = 0; q3 < nk[2]; ++q3)
        for (int q2 = 0; q2 < nk[1]; ++q2)
            for (int q1 = 0; q1 < nk[0]; ++q1)
                TQ[((size_t)q1 * nk[1] + q2) * nk[2] + q3] = T[((size_t)q3 * nk[1] + q2) * nk[0] + q1];

    chasm_theta_s* h = new (std::nothrow) chasm_theta_s();
    if (!h) return tfail(CHASM_ENOMEM, "host allocation failed");
    h->desc = *desc;
    h->stream = (hipStream_t)hip_stream;
    h->ks = ks;
    h->npts = (long long)desc->nx[0] * desc->nx[1] * desc->nx[2];
    h->nkp = (long long)nk[0] * nk[1] * nk[2];
    auto bail = [&](chasm_status s, const std::string& m) {
        chasm_theta_destroy(h);
        (void)hipGetLastError();   // reported by this call, not by the next launch of another handle
        return tfail(s, m);
    };
    h->plan = theta_plan(desc, ks);
    if (hipMalloc((void**)&h->T, TQ.size() * sizeof(double)) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(tensor) failed");
    if (hipMemcpyAsync(h->T, TQ.data(), TQ.size() * sizeof(double), hipMemcpyHostToDevice, h->stream) != hipSuccess)
        return bail(CHASM_EDEVICE, "tensor upload failed");
    const size_t es = desc->dtype == CHASM_F64 ? 8 : 4;
    if (hipMalloc(&h->ws, (size_t)h->npts * h->nkp * desc->nbatch * es) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(workspace) failed");
    if (hipMalloc((void**)&h->tab, h->plan.tab) != hipSuccess || hipMalloc((void**)&h->U, h->plan.U) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(kernel tables) failed");
    if (h->plan.W && hipMalloc((void**)&h->W, h->plan.W) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(staged intermediate) failed");
    ThetaArgs& a = h->args;
    a.npts = h->npts;
    a.nnuc = desc->nnuc;
    a.nbatch = desc->nbatch;
    const double PP = 4.0 * nk[0] * nk[1];
    for (int d = 0; d < 3; ++d) {
        a.nx[d] = desc->nx[d];
        a.x_lo[d] = desc->x_lo[d];
        a.hx[d] = (desc->x_hi[d] - desc->x_lo[d]) / desc->nx[d];
        a.hk[d] = hk[d];
    }
    for (int i = 0; i < desc->nnuc; ++i) {
        for (int d = 0; d < 3; ++d) a.xa[i][d] = desc->x_nuc[i][d];
        a.wgt[i] = desc->z_nuc[i] * (2.0 / (M_PI * M_PI)) / (2.0 * PP);   // z_a 4/c_{3,1}, c_{3,1} = 2 pi^2; 1/P^2 of the inverse
    }
    if (hipMalloc((void**)&h->et, (size_t)mod_rows(a) * nk[0] * sizeof(fft::cd)) != hipSuccess)
        return bail(CHASM_ENOMEM, "hipMalloc(factors) failed");
    if (ks->mod(h->et, a, h->stream) != hipSuccess) return bail(CHASM_EDEVICE, "factors launch failed");
    if (h->plan.u_resident && ks->node(h->U, h->T, h->et, a, 0, desc->nx[0], h->stream) != hipSuccess)
        return bail(CHASM_EDEVICE, "kernel table launch failed");
    if (h->plan.resident && make_tables(h, ThetaRange{0, 0, 0, h->plan.np}) != hipSuccess)
        return bail(CHASM_EDEVICE, "kernel table launch failed");
    if (hipStreamSynchronize(h->stream) != hipSuccess) return bail(CHASM_EDEVICE, "stream synchronize failed");
    *out = h;
    return CHASM_OK;
}

chasm_status chasm_theta_apply(chasm_theta_t h, const void* f_dev, void* out_dev)
{
    if (!h || !f_dev || !out_dev) return tfail(CHASM_EINVAL, "NULL argument");
    if (h->poisoned) return tfail(CHASM_ESTATE, "handle is poisoned by an earlier device failure");
    return run_theta(h, TR_PLAIN, f_dev, nullptr, 0.0, TR_PLAIN, out_dev, nullptr, 0.0);
}

chasm_status chasm_theta_destroy(chasm_theta_t h)
{
    if (!h) return CHASM_OK;
    if (h->stream) hipStreamSynchronize(h->stream);
    if (h->T) hipFree(h->T);
    if (h->tab) hipFree(h->tab);
    if (h->U) hipFree(h->U);
    if (h->et) hipFree(h->et);
    if (h->ws) hipFree(h->ws);
    if (h->W) hipFree(h->W);
    delete h;
    return CHASM_OK;
}

}  // extern "C"
