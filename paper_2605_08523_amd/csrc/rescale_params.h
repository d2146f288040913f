// The rescale of Sec. IV.1 from the Gershgorin bounds (Eqs. mu', beta', flip, conditions), in FP64.
#pragma once

#include <math.h>

#include "fe_internal.h"

namespace fe {

__device__ inline Params rescale_params(double lo, double hi, int bad, double mu, double kT,
                                        double beta0, double mu0) {
    Params p;
    p.emin = lo;
    p.emax = hi;
    p.flipped = 0;
    p.clamped = 0;
    p.degenerate = 0;
    p.status = FE_OK;
    const double width = hi - lo;
    if (bad || !isfinite(lo) || !isfinite(hi)) {
        p.status = FE_ERR_NONFINITE;
        p.mu_p = p.beta_p = p.beta_max = NAN;
        p.scale = p.shift = NAN;
    } else if (width <= 1e-300 * fmax(1.0, fabs(hi))) {
        // H = c I: the model coordinate of every eigenvalue is y = mu0 + (mu - c)/(kT beta0).
        double y = mu0 + (mu - lo) / (kT * beta0);
        p.degenerate = 1;
        if (!(y >= 0.0 && y <= 1.0)) {
            p.clamped = 1;
            y = fmin(1.0, fmax(0.0, y));
        }
        p.mu_p = NAN;
        p.beta_p = INFINITY;
        p.beta_max = NAN;
        p.scale = 0.0;
        p.shift = y;
    } else if (!(lo < mu && mu < hi)) {
        p.status = FE_ERR_DOMAIN;
        p.mu_p = p.beta_p = p.beta_max = NAN;
        p.scale = p.shift = NAN;
    } else {
        double mu_p = (hi - mu) / width;           // Eq. mu'
        double beta_p = width / kT;                // Eq. beta'
        const int flip = mu_p > 0.5;               // Eq. flip (strict)
        if (flip) mu_p = 1.0 - mu_p;
        const double bmax = fmin(mu0 / mu_p, (1.0 - mu0) / (1.0 - mu_p)) * beta0;  // Eq. conditions
        if (beta_p > bmax) {
            beta_p = bmax;
            p.clamped = 1;
            p.status = FE_WARN_BETA_CLAMPED;
        }
        const double r = beta_p / beta0;
        // X0 = r (H' - mu' I) + mu0 I with H' = (emax I - H)/width, or its flip (H - emin I)/width.
        p.scale = flip ? r / width : -r / width;
        p.shift = flip ? r * (-lo / width - mu_p) + mu0 : r * (hi / width - mu_p) + mu0;
        p.mu_p = mu_p;
        p.beta_p = beta_p;
        p.beta_max = bmax;
        p.flipped = flip;
    }
    return p;
}

}  // namespace fe
