// resident.h -- evaluations and inversions of small boxes in one workgroup per replica.
#pragma once

#include "hsf_internal.h"

namespace hsf {

constexpr int kResZ = 4;   // planes of a thread's column

enum { RES_EVAL = 0, RES_START = 1, RES_PASSES = 2 };

// Whether every replica is at most 16 x 16 x 16 (and its two propagators fit the LDS).
bool resident_fits(const Rep *reps, int n_rep, size_t real_bytes, size_t lds_limit);

template <typename real>
hipError_t launch_resident(hipStream_t s, int kind, const Rep *reps_host, int n_rep, const Rep *rep, RepState *st,
                           const Chain &ch, real *G, double *w, double *d, const double *phi, double *out, double tol,
                           int max_iter, int max_passes, RepState *mirror);

}  // namespace hsf
