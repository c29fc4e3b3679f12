// C ABI of the OC update (arXiv 2505.02438, Sec. 2.3, Algorithm 1); the
// kernels are in oc.hip.  The host launches a search for the multiplier and a
// proof of the bisection's path to it; where that form does not apply or the
// proof fails, it launches bisection passes (each advances up to kOcDepth
// steps on the device) in batches and reads the done flag after each batch.
#include <hip/hip_runtime.h>

#include <cmath>

#include "../../include/soptx_debug.h"
#include "../../include/soptx_oc.h"
#include "host_util.h"
#include "internal.h"
#include "kernels.h"

using namespace soptx;

namespace {
constexpr int kPassesPerCheck = 4;
constexpr double kDirectTol = 1e-5;
thread_local int t_last_form = -1;  // soptx_debug_oc_form
}

extern "C" int soptx_debug_oc_form(int32_t *form) {
    if (!form) return SOPTX_E_INVALID_ARG;
    *form = t_last_form;
    return SOPTX_OK;
}

extern "C" int soptx_oc_update(int64_t n, const double *d_rho, const double *d_dc, const double *d_dv,
                               double vol_target, const soptx_oc_params *prm, double *d_rho_new,
                               soptx_oc_result *out, void *stream) {
    if (!prm || !out || n < 0 || !std::isfinite(vol_target)) return SOPTX_E_INVALID_ARG;
    if (!(prm->move > 0.0 && prm->move <= 1.0) || !(prm->eta > 0.0 && prm->eta <= 1.0) ||
        !(prm->lmax > 0.0 && std::isfinite(prm->lmax)) || !(prm->tol > 0.0 && prm->tol < 1.0) ||
        prm->max_steps < 1 || prm->max_steps > 1000)
        return SOPTX_E_INVALID_ARG;
    *out = soptx_oc_result{0.0, 0.0, 0.0, 0};
    t_last_form = -1;
    if (n == 0) return SOPTX_OK;
    if (!d_rho || !d_dc || !d_dv || !d_rho_new || d_rho_new == d_rho || d_rho_new == d_dc || d_rho_new == d_dv)
        return SOPTX_E_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return SOPTX_E_DEVICE;
    double *ws = nullptr;
    int rc = get_workspace(dev, st, (size_t)kOcNodes * kOcMaxBlocks + 8 + kOcSlots + kOcAcc, &ws, 3);
    if (rc) return rc;
    double *state = ws, *part = ws + 8 + kOcSlots, *acc = part + kOcNodes * kOcMaxBlocks;
    double h[8 + kOcSlots];
    auto read_state = [&]() {
        return hipMemcpyAsync(h, state, sizeof(h), hipMemcpyDeviceToHost, st) == hipSuccess &&
               hipStreamSynchronize(st) == hipSuccess;
    };
    auto result = [&]() {
        out->lambda = h[2];
        out->volume = h[3];
        out->steps = (int32_t)h[4];
        out->change = h[6];
        return SOPTX_OK;
    };
    if (launch_oc_init(state, prm->lmax, acc, st) != hipSuccess) return SOPTX_E_DEVICE;
    // Search and proof where the update's operations are correctly rounded
    // (eta 0.5 or 1) and the final bracket is wide against the search's
    // accuracy (about 1e-7: a tighter one would seldom be proved).
    if ((prm->eta == 0.5 || prm->eta == 1.0) && prm->tol >= kDirectTol) {
        if (launch_oc_direct(d_rho, d_dc, d_dv, n, prm->move, prm->eta, vol_target, prm->lmax, prm->tol,
                             prm->max_steps, state, acc, part, d_rho_new, st) != hipSuccess ||
            !read_state())
            return SOPTX_E_DEVICE;
        if (h[5] != 0.0) {
            for (int k = 0; k < kOcSlots; k++)  // all are 0, positive or NaN: a NaN stays
                if (h[8 + k] > h[6] || std::isnan(h[8 + k])) h[6] = h[8 + k];
            t_last_form = 1;
            return result();
        }
        if (launch_oc_init(state, prm->lmax, acc, st) != hipSuccess) return SOPTX_E_DEVICE;
    }
    const int max_passes = (prm->max_steps + kOcDepth - 1) / kOcDepth;
    for (int p = 0; p < max_passes;) {
        for (int q = 0; q < kPassesPerCheck && p < max_passes; q++, p++)
            if (launch_oc_pass(d_rho, d_dc, d_dv, n, prm->move, prm->eta, vol_target, prm->tol, prm->max_steps,
                               state, part, st) != hipSuccess)
                return SOPTX_E_DEVICE;
        if (!read_state()) return SOPTX_E_DEVICE;
        if (h[5] != 0.0) break;
    }
    if (launch_oc_apply(d_rho, d_dc, d_dv, n, prm->move, prm->eta, state, d_rho_new, part, st) != hipSuccess)
        return SOPTX_E_DEVICE;
    if (!read_state()) return SOPTX_E_DEVICE;
    t_last_form = 0;
    return result();
}
