// chasm_lpc1.hip -- the LPC1 time step (Sec. 2.2) built from the characteristic step
// (chasm_advect.h) and the truncated-kernel Theta_V (chasm_theta.h).  See
// include/chasm_lpc1.h.
//
// State: the caller's field f and the library's field G.  One step:
//   G = Theta[f]                (theta apply, f -> G)
//   f = A f,  G = A G           (two advection handles on the same stream, one per field)
//   f = f + tau/2 (G + Theta[f + tau G])
// The predictor f + tau G is formed while the operator's first transpose reads the two
// fields, the corrector while its last one writes (theta_lpc1), so neither is a pass of
// its own and the predictor needs no field: on 61^3 x 16^3 FP32 the two transposes take
// 2.3 and 3.1 ms, against 1.3 each and 5.3 ms for two combination passes.  f is stepped in place, so no step copies
// the field in or out.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <string>

#include "../../include/chasm_lpc1.h"

namespace chasm {
void set_last_error(const std::string& msg);

chasm_status theta_lpc1(chasm_theta_t h, void* f, const void* g, double tau);   // chasm_theta.hip

}  // namespace chasm

using namespace chasm;

struct chasm_lpc1_s {
    chasm_advect_t adv_f = nullptr;   // characteristic step of the caller's field
    chasm_advect_t adv_g = nullptr;   // characteristic step of G
    chasm_theta_t th = nullptr;
    void* f = nullptr;          // caller's field
    void* G = nullptr;          // [field]: Theta[f^n], then A Theta[f^n]
    hipStream_t stream = nullptr;
    int dtype = 0;
    double tau = 0.0;
    bool poisoned = false;
};

static chasm_status lfail(chasm_status st, const std::string& m)
{
    set_last_error(m);
    return st;
}

extern "C" {

chasm_status chasm_lpc1_create(const chasm_advect_desc* adv, const chasm_theta_desc* th, void* f_dev,
                               void* hip_stream, chasm_lpc1_t* out)
{
    if (!out) return lfail(CHASM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!adv || !th || !f_dev) return lfail(CHASM_EINVAL, "NULL argument");
    if (adv->nbatch != 1 || th->nbatch != 1) return lfail(CHASM_EINVAL, "LPC1 steps one field (nbatch 1)");
    if (adv->flags != 0) return lfail(CHASM_EINVAL, "advection flags must be 0 for LPC1");
    if (adv->dtype != th->dtype) return lfail(CHASM_EINVAL, "advection and theta dtypes differ");
    for (int a = 0; a < 3; ++a)
        if (adv->nx[a] != th->nx[a] || adv->nk[a] != th->nk[a] || adv->x_lo[a] != th->x_lo[a] ||
            adv->x_hi[a] != th->x_hi[a] || adv->k_lo[a] != th->k_lo[a] || adv->k_hi[a] != th->k_hi[a])
            return lfail(CHASM_EINVAL, "advection and theta grids differ");
    if (!(adv->dt > 0) || !std::isfinite(adv->dt)) return lfail(CHASM_EINVAL, "tau (adv->dt) must be finite and > 0");

    chasm_lpc1_s* h = new (std::nothrow) chasm_lpc1_s();
    if (!h) return lfail(CHASM_ENOMEM, "host allocation failed");
    h->f = f_dev;
    h->stream = (hipStream_t)hip_stream;
    h->dtype = adv->dtype;
    h->tau = adv->dt;
    long long n = 1;            // values per field
    for (int a = 0; a < 3; ++a) n *= (long long)adv->nx[a] * adv->nk[a];
    const size_t bytes = (size_t)n * (h->dtype == CHASM_F64 ? 8 : 4);
    auto bail = [&](chasm_status s, const std::string& m) {
        chasm_lpc1_destroy(h);
        (void)hipGetLastError();   // reported by this call, not by the next launch of another handle
        return lfail(s, m);
    };
    if (hipMalloc(&h->G, bytes) != hipSuccess) return bail(CHASM_ENOMEM, "hipMalloc(theta field) failed");
    chasm_status st = chasm_advect_create(adv, f_dev, hip_stream, &h->adv_f);
    if (st == CHASM_OK) st = chasm_advect_create(adv, h->G, hip_stream, &h->adv_g);
    if (st != CHASM_OK) {
        const std::string m = chasm_advect_last_error();
        return bail(st, "advection: " + m);
    }
    st = chasm_theta_create(th, hip_stream, &h->th);
    if (st != CHASM_OK) {
        const std::string m = chasm_advect_last_error();
        return bail(st, "theta: " + m);
    }
    *out = h;
    return CHASM_OK;
}

chasm_status chasm_lpc1_step(chasm_lpc1_t h, int32_t nsteps)
{
    if (!h) return lfail(CHASM_EINVAL, "handle is NULL");
    if (h->poisoned) return lfail(CHASM_ESTATE, "handle is poisoned by an earlier device failure");
    if (nsteps < 0) return lfail(CHASM_EINVAL, "nsteps must be >= 0");
    if (nsteps == 0) return CHASM_OK;
    for (int s = 0; s < nsteps; ++s) {
        chasm_status st = chasm_theta_apply(h->th, h->f, h->G);
        if (st == CHASM_OK) st = chasm_advect_step(h->adv_f, 1);
        if (st == CHASM_OK) st = chasm_advect_step(h->adv_g, 1);
        if (st == CHASM_OK) st = theta_lpc1(h->th, h->f, h->G, h->tau);
        if (st != CHASM_OK) {
            h->poisoned = true;
            return st;
        }
    }
    return CHASM_OK;
}

chasm_status chasm_lpc1_destroy(chasm_lpc1_t h)
{
    if (!h) return CHASM_OK;
    if (h->stream) hipStreamSynchronize(h->stream);
    if (h->adv_f) chasm_advect_destroy(h->adv_f);
    if (h->adv_g) chasm_advect_destroy(h->adv_g);
    if (h->th) chasm_theta_destroy(h->th);
    if (h->G) hipFree(h->G);
    delete h;
    return CHASM_OK;
}

}  // extern "C"
