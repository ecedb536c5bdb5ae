// ctl_device.h -- the scalar logic of the Fletcher-Reeves inversion of one replica (the steps
// are described in ctl.hip), shared by the control kernel and the resident kernels.
#pragma once

#include <math.h>

#include "device_common.h"

namespace hsf {

// Nearest integer to log2(m), m > 0 finite, from the binary exponent.
__device__ __forceinline__ long round_log2(double m)
{
    int e = 0;
    const double f = frexp(m, &e);   // m = f 2^e, f in [0.5, 1)
    return f < 0.70710678118654752440 ? e - 1 : e;
}

// Per-step power-of-two scales for the next evaluation.  sums[s] = sum_r of the
// stored G_{s+1} of this evaluation (its mean m_s is relative to the cumulative
// scale used), sums[N], sums[N+1] = sum_r E_A, E_B.  Target: stored means near 1.
// Where a mean is not usable (overflow or underflow) the growth is predicted from
// the mean-field factor <E_{t_s}> csum instead.
__device__ inline void update_scales(RepState &S, const Chain &ch, const double *sums, double V, double csum)
{
    int cum_old = 0, cum_new = 0;
    for (int s = 0; s < ch.N; ++s) {
        cum_old += S.scale_e[s];
        const double m = sums[s] / V;
        long target;
        if (m > 0.0 && isfinite(m)) {
            target = cum_old + round_log2(m);
        } else {
            const double me = sums[ch.N + ch.types[s]] / V * csum;
            target = cum_new + ((me > 0.0 && isfinite(me)) ? round_log2(me) : 0);
        }
        long e = target - cum_new;
        if (e > 100) e = 100;
        if (e < -100) e = -100;
        S.scale_e[s] = (int)e;
        cum_new += (int)e;
    }
}

// Scalar logic of one replica after the reductions of a phase (runs in one thread).
__device__ inline void control(RepState &S, int phase, const Chain &ch, const double *red, const double *gsum,
                        double V, double csum, double tol, int max_iter)
{
    switch (phase) {
    case PH_Q: {
        bool bad;
        q_from_sum(gsum[ch.N - 1], V, S.scale_e, ch.N, S.q, S.ln_q, bad);
        if (bad) S.nonfinite = 1;
        break;
    }
    case PH_TARGET_SOLVENT: S.sol_mean = red[6] / V; [[fallthrough]];
    case PH_TARGET: {
        S.phibar_p = red[0] / V;
        S.phibar_s = red[1] / V;
        S.tnorm2[0] = red[2];
        S.tnorm2[1] = red[3];
        S.wmean[0] = red[4] / V;
        S.wmean[1] = red[5] / V;
        S.tol = tol;
        S.max_iter = max_iter;
        S.active = 1;
        S.done = 0;
        S.pending = 0;
        S.accepted = 0;
        S.iters = 0;
        S.evals = 0;
        S.restarts = 0;
        S.converged = 0;
        S.nonfinite = 0;
        S.trial = 0;
        S.alpha = 0.0;
        S.res = INFINITY;
        break;
    }
    case PH_SCALES: update_scales(S, ch, gsum, V, csum); break;
    case PH_EVAL0: {
        update_scales(S, ch, gsum, V, csum);
        S.evals += 1;
        S.gg = red[1];
        S.res = fmax(sqrt(red[2] / S.tnorm2[0]), sqrt(red[3] / S.tnorm2[1]));
        S.active = 0;
        if (!isfinite(S.res) || S.nonfinite) {
            S.nonfinite = 1;
            S.done = 1;
        } else if (S.res <= S.tol) {
            S.done = 1;
            S.converged = 1;
        } else if (S.max_iter <= 0) {
            S.done = 1;
        } else {
            S.pending = 1;
        }
        break;
    }
    case PH_BEGIN: {
        S.h0 = red[0];
        S.dhd = red[1];
        S.alpha = -S.h0 / S.dhd;
        S.a_prev = 0.0;
        S.h_prev = S.h0;
        S.trial = 1;
        S.active = 1;
        S.accepted = 0;
        S.pending = 0;
        if (!isfinite(S.alpha)) {
            S.nonfinite = 1;
            S.done = 1;
            S.active = 0;
        }
        break;
    }
    case PH_TRIAL: {
        S.evals += 1;
        const double h = red[0];
        bool accept = fabs(h) <= 0.1 * fabs(S.h0) || S.trial >= 3;
        if (!accept) {
            const double slope = (h - S.h_prev) / (S.alpha - S.a_prev);
            if (!(slope > 0.0)) {
                accept = true;
            } else {
                double an = S.alpha - h / slope;
                if (!(an > 0.0)) {
                    accept = true;
                } else {
                    if (an > 8.0 * S.alpha) an = 8.0 * S.alpha;
                    S.a_prev = S.alpha;
                    S.h_prev = h;
                    S.alpha = an;
                    S.trial += 1;
                }
            }
        }
        if (accept) {
            S.active = 0;
            S.accepted = 1;
            S.iters += 1;
            S.res = fmax(sqrt(red[2] / S.tnorm2[0]), sqrt(red[3] / S.tnorm2[1]));
            if (!isfinite(S.res) || S.nonfinite) {
                S.nonfinite = 1;
                S.done = 1;
                S.beta = 0.0;
            } else if (S.res <= S.tol) {
                S.converged = 1;
                S.done = 1;
                S.beta = 0.0;
            } else {
                const double ggn = red[1];
                double beta = ggn / S.gg;
                S.gg = ggn;
                if (S.iters % 50 == 0) {
                    beta = 0.0;
                    S.restarts += 1;
                } else if (-ggn + beta * h >= 0.0) {
                    beta = 0.0;
                    S.restarts += 1;
                }
                S.beta = beta;
                if (S.iters >= S.max_iter) {
                    S.done = 1;
                } else {
                    S.pending = 1;
                }
            }
        }
        break;
    }
    default: break;
    }
}

}  // namespace hsf
