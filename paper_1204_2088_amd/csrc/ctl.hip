// ctl.hip -- deterministic reductions and the per-replica control of the
// Fletcher-Reeves inversion (section 2: the fields are determined
// self-consistently at every step by nonlinear conjugate gradients).
//
// The inversion minimises the convex objective
//   Phi(w) = (phibar_p V / N) ln Q[w] + phibar_s V ln<exp(-w_S)> + sum_I sum_r phi^t_I w_I,
// whose gradient is phi^t - phi[w].  Line search: secant on h(alpha) = d.grad Phi(w + alpha d)
// from alpha_0 = -(d.g) / sum d^2 phi^t; a trial is accepted when |h| <= 0.1 |h(0)|, after
// three trials, or when the secant slope or the next alpha is not positive (extrapolation
// capped at 8x).  beta = (g_new.z_new) / (g_old.z_old) with z = g, or z = g / phi^t in the
// diagonally preconditioned variant; restart every 50 iterations and whenever the new
// direction would not descend (d_new.g_new = -g_new.z_new + beta d.g_new >= 0).
//
// All vector work is done by site kernels that write per-block partial sums; one block
// per replica then sums its blocks' partials in a fixed order and thread 0 runs the
// replica's scalar logic, so every replica of a batch follows its own iteration.
#include <math.h>

#include "ctl_device.h"

namespace hsf {

__device__ void reduce_and_control(RepState &S, int r, const int *__restrict__ blk_first, const Rep *__restrict__ rep,
                                   const double *__restrict__ part, int phase, const Chain &ch,
                                   const int *__restrict__ gblk_first, const double *__restrict__ partG, int nblocks,
                                   double tol, int max_iter);

// One workgroup of kCtlBlock threads per replica: its reductions are chains of dependent
// load batches, so more wavefronts per row shorten them.
constexpr int kCtlBlock = 1024;

__global__ __launch_bounds__(kCtlBlock) void k_reduce_ctl(const int *__restrict__ blk_first,
                                                       RepState *__restrict__ st, const Rep *__restrict__ rep,
                                                       const double *__restrict__ part, int phase, Chain ch,
                                                       const int *__restrict__ gblk_first,
                                                       const double *__restrict__ partG, int nblocks,
                                                       double tol, int max_iter, RepState *__restrict__ mirror)
{
    const int r = blockIdx.x;
    // work on an LDS copy of the replica's state: one cooperative load and store instead of
    // a dependent global round trip per field in the scalar logic below
    __shared__ RepState S;
    {
        static_assert(sizeof(RepState) % 4 == 0, "RepState is copied as 32-bit words");
        const int *src = reinterpret_cast<const int *>(&st[r]);
        int *dst = reinterpret_cast<int *>(&S);
        for (int k = threadIdx.x; k < (int)(sizeof(RepState) / 4); k += kCtlBlock) dst[k] = src[k];
    }
    __syncthreads();

    // which replicas take part in this phase (uniform per block)
    bool take;
    switch (phase) {
    case PH_Q: case PH_EVAL0: case PH_TRIAL: case PH_SCALES: take = S.active != 0; break;
    default: take = true; break;
    }
    if (take && phase == PH_BEGIN && !S.pending) {
        take = false;
        __syncthreads();
        if (threadIdx.x == 0) S.accepted = 0;
    }
    if (take) reduce_and_control(S, r, blk_first, rep, part, phase, ch, gblk_first, partG, nblocks, tol, max_iter);
    __syncthreads();
    {
        // the state back to device memory and into the host's pinned mirror, which the
        // host reads after synchronising the stream (no copy launch)
        const int *src = reinterpret_cast<const int *>(&S);
        int *dst = reinterpret_cast<int *>(&st[r]);
        int *hm = mirror ? reinterpret_cast<int *>(&mirror[r]) : nullptr;
        for (int k = threadIdx.x; k < (int)(sizeof(RepState) / 4); k += kCtlBlock) {
            dst[k] = src[k];
            if (hm) hm[k] = src[k];
        }
    }
}

// The reduction of one phase's partial sums for replica r and the scalar control step.
__device__ void reduce_and_control(RepState &S, int r, const int *__restrict__ blk_first, const Rep *__restrict__ rep,
                                   const double *__restrict__ part, int phase, const Chain &ch,
                                   const int *__restrict__ gblk_first, const double *__restrict__ partG, int nblocks,
                                   double tol, int max_iter)
{
    const int b0 = blk_first[r], b1 = blk_first[r + 1];
    const int gb0 = gblk_first[r], gb1 = gblk_first[r + 1];
    const double V = (double)rep[r].V;
    __shared__ double vals[kNQ + 66];

    // rows to reduce: nslots slots of `part`, then ng rows of `partG` starting at g_first
    int nslots = 0, g_first = 0, ng = 0;
    switch (phase) {
    case PH_TARGET: nslots = 6; break;
    case PH_TARGET_SOLVENT: nslots = 7; break;
    case PH_EVAL0: nslots = 4; ng = ch.N + 2; break;
    case PH_TRIAL: nslots = 4; break;
    case PH_SCALES: ng = ch.N + 2; break;
    case PH_Q: g_first = ch.N - 1; ng = 1; break;
    case PH_BEGIN: nslots = 2; break;
    default: break;
    }
    // Each row is split into contiguous parts of the replica's blocks, one wavefront per
    // part (as many parts as the wavefronts allow, the same for every row of the phase);
    // within a part the lanes stride over the blocks and a fixed order adds them,
    // then the parts are added in order: the order of additions is fixed, so results are
    // reproducible.
    constexpr int kWaves = kCtlBlock / 64;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int nrows = nslots + ng;
    const int parts = nrows > 0 ? (nrows >= kWaves ? 1 : kWaves / nrows) : 1;
    __shared__ double psum[kWaves];
    for (int t0 = 0; t0 < nrows * parts; t0 += kWaves) {
        const int t = t0 + wid, row = t / parts, pt = t % parts;
        if (row < nrows) {
            // `part` has a slot per block of the density launch, partG a column per block of
            // the forward sweep (another plan when the sweeps have their own tiles)
            const int f0 = row < nslots ? b0 : gb0, f1 = row < nslots ? b1 : gb1;
            const int span = (f1 - f0 + parts - 1) / parts;
            const int lo = f0 + pt * span, hi = lo + span < f1 ? lo + span : f1;
            double v = 0.0;
            // unrolled so that the loads of several iterations are in flight together
            if (row < nslots) {
#pragma unroll 8
                for (int b = lo + lane; b < hi; b += 64) v += part[(long long)b * kNQ + row];
            } else {
                const double *base = partG + (long long)(g_first + row - nslots) * nblocks;
#pragma unroll 8
                for (int b = lo + lane; b < hi; b += 64) v += base[b];
            }
            v = wave_sum(v);
            if (lane == 0) psum[wid] = v;
        }
        __syncthreads();
        // the rows completed in this round: their parts are the wavefronts t0 .. t0 + kWaves
        if (threadIdx.x < kWaves / parts) {
            const int row = t0 / parts + threadIdx.x;
            if (row < nrows) {
                double v = 0.0;
                for (int q = 0; q < parts; ++q) v += psum[threadIdx.x * parts + q];
                vals[row] = v;
            }
        }
        __syncthreads();
    }
    const double *red = vals;
    const double *gsum = vals + nslots - g_first;   // gsum[s] = sum of stored G_{s+1}
    if (threadIdx.x == 0) control(S, phase, ch, red, gsum, V, rep[r].csum, tol, max_iter);
}

void launch_reduce_ctl(hipStream_t s, int n_rep, const Plan &p, RepState *st, const Rep *rep,
                       const double *part, int phase, Chain ch, const Plan &pg, const double *partG, double tol,
                       int max_iter, RepState *mirror)
{
    hipLaunchKernelGGL(k_reduce_ctl, dim3(n_rep), dim3(kCtlBlock), 0, s, p.blk_first, st, rep, part, phase, ch,
                       pg.blk_first, partG, pg.nblocks, tol, max_iter, mirror);
}

// Partial sums of the inversion target: sum of polymer phi^t, sum of phi^t_S,
// |phi^t_A|^2, |phi^t_B|^2, sum of w_A and of w_B, and (SOLVENT) of exp(-w_S).  One read of
// the arrays; a block takes p.span sites, so that its reduction of seven sums and the
// control kernel's pass over the blocks are paid once per span (128^3: 30.5 us for 8192
// blocks of 256 sites and 11 us in the control kernel).  E (or null): also the polymers' field
// factors exp(-w), as launch_field_exp writes them, from the same read of w.
// Bound by its loads: those of four sites are issued together, unconditionally (128^3 solution,
// FP32 with field factors: 24.4 us in a kernel trace, 118 MB at 4.8 TB/s, the rate of a copy; 32.7 with a
// bounds test between the sites, which left one site's loads in flight).
template <bool SOLVENT, typename real>
__global__ __launch_bounds__(kBlock) void k_target_stats(const int *__restrict__ blk_rep,
                                                         const int *__restrict__ blk_first,
                                                         const Rep *__restrict__ rep, int nsp, int span,
                                                         const double *__restrict__ phit,
                                                         const double *__restrict__ w, double *__restrict__ part,
                                                         real *__restrict__ E)
{
    const SiteRef sr = span_ref(blk_rep, blk_first, span);
    const Rep &R = rep[sr.r];
    const long long V = R.V;
    const long long fo = off_field(R, nsp), po = off_poly(R);
    constexpr int NV = SOLVENT ? 7 : 6;
    double v[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = 0.0;
    constexpr int U = 4;   // sites whose loads are in flight together
    for (int u0 = 0; u0 < span; u0 += U * kBlock) {
        const int n = min(U, (span - u0) / kBlock);
        double a[U], b[U], c[U], wa[U], wb[U], ws[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const long long i = min(sr.i + u0 + min(k, n - 1) * kBlock, V - 1);
            a[k] = phit[fo + i];
            b[k] = phit[fo + V + i];
            c[k] = nsp == 3 ? phit[fo + 2 * V + i] : 0.0;
            wa[k] = w[fo + i];
            wb[k] = w[fo + V + i];
            ws[k] = SOLVENT ? w[fo + 2 * V + i] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const long long i = sr.i + u0 + k * kBlock;
            if (k >= n || i >= V) continue;
            v[0] += a[k] + b[k];
            v[1] += c[k];
            v[2] += a[k] * a[k];
            v[3] += b[k] * b[k];
            v[4] += wa[k];
            v[5] += wb[k];
            if (E) {
                E[po + i] = (real)exp(-wa[k]);
                E[po + V + i] = (real)exp(-wb[k]);
            }
            if (SOLVENT) v[NV - 1] += exp(-ws[k]);
        }
    }
    block_sums(v);
    if (threadIdx.x == 0)
        for (int q = 0; q < NV; ++q) part[(long long)plan_block() * kNQ + q] = v[q];
}

template <typename real>
void launch_target_stats(hipStream_t s, const Plan &p, const Rep *rep, Chain ch, const double *phit, const double *w,
                         bool solvent, double *part, real *E)
{
    auto kern = solvent ? k_target_stats<true, real> : k_target_stats<false, real>;
    hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, ch.nsp, p.span, phit, w,
                       part, E);
}
template void launch_target_stats<float>(hipStream_t, const Plan &, const Rep *, Chain, const double *, const double *,
                                         bool, double *, float *);
template void launch_target_stats<double>(hipStream_t, const Plan &, const Rep *, Chain, const double *, const double *,
                                          bool, double *, double *);

// Local ideal-gas starting guess w_I = -ln phi_I (the constant -ln <phi_I> is removed
// by the gauge shift that follows).
__global__ __launch_bounds__(kBlock) void k_local_guess(const int *__restrict__ blk_rep,
                                                        const int *__restrict__ blk_first,
                                                        const Rep *__restrict__ rep, Chain ch,
                                                        const double *__restrict__ phit, double *__restrict__ w)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    const long long fo = off_field(R, ch.nsp);
    for (int I = 0; I < 2; ++I) w[fo + I * V + i] = -log(phit[fo + I * V + i]);
}

void launch_local_guess(hipStream_t s, const Plan &p, const Rep *rep, Chain ch, const double *phit,
                        double *w, double *)
{
    hipLaunchKernelGGL(k_local_guess, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, ch,
                       phit, w);
}

// Gauge shift of the polymer fields to zero mean; closed-form solvent field
// w_S = -ln(phi^t_S / phibar_s).
__global__ __launch_bounds__(kBlock) void k_init_fields(const int *__restrict__ blk_rep,
                                                        const int *__restrict__ blk_first,
                                                        const Rep *__restrict__ rep, const RepState *__restrict__ st,
                                                        Chain ch, const double *__restrict__ phit,
                                                        double *__restrict__ w)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    const RepState &S = st[sr.r];
    const long long fo = off_field(R, ch.nsp);
    w[fo + i] -= S.wmean[0];
    w[fo + V + i] -= S.wmean[1];
    if (ch.nsp == 3) w[fo + 2 * V + i] = -log(phit[fo + 2 * V + i] / S.phibar_s);
}

void launch_init_fields(hipStream_t s, const Plan &p, const Rep *rep, RepState *st, Chain ch,
                        const double *phit, double *w)
{
    hipLaunchKernelGGL(k_init_fields, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, st, ch,
                       phit, w);
}

// Conjugate-gradient vector update, z = g (or g / phi^t when preconditioned).
//   init = 1 (replicas pending their first iteration): d = -z, g from the start evaluation
//   init = 0 (replicas whose trial was accepted): w += alpha d and, unless the replica is
//            done, d = -z + beta d with g the accepted trial's gradient g_trial (read in
//            place: only the scalars of g are needed later, and the next start evaluation
//            rewrites the vector g)
// Partial sums d.g and sum d^2 phi^t for the next alpha_0.
__global__ __launch_bounds__(kBlock) void k_cg_update(const int *__restrict__ blk_rep,
                                                      const int *__restrict__ blk_first,
                                                      const Rep *__restrict__ rep, const RepState *__restrict__ st,
                                                      int nsp, int precond, int span, int init,
                                                      double *__restrict__ w, const double *__restrict__ g,
                                                      const double *__restrict__ gt, double *__restrict__ d,
                                                      const double *__restrict__ phit, double *__restrict__ part)
{
    const SiteRef sr = span_ref(blk_rep, blk_first, span);
    const RepState &S = st[sr.r];
    if (init ? !S.pending : !S.accepted) return;
    const Rep &R = rep[sr.r];
    const long long V = R.V;
    const long long fo = off_field(R, nsp), po = off_poly(R);
    const double alpha = S.alpha, beta = S.beta;
    const bool upd_d = init || !S.done;
    const double *gs = init ? g : gt;
    double t[2] = {0.0, 0.0};
#pragma unroll 2
    for (int u = 0; u < span; u += kBlock) {
        const long long i = sr.i + u;
        if (i >= V) break;
#pragma unroll
        for (int I = 0; I < 2; ++I) {
            const long long k = po + I * V + i, kf = fo + I * V + i;
            double dI = d[k];
            const double gI = gs[k], pI = phit[kf];
            if (!init) w[kf] = fma(alpha, dI, w[kf]);
            if (upd_d) {
                const double zI = precond ? gI / pI : gI;
                dI = init ? -zI : fma(beta, dI, -zI);
                d[k] = dI;
            }
            t[0] += dI * gI;
            t[1] += dI * dI * pI;
        }
    }
    block_sums(t);
    if (threadIdx.x == 0) {
        part[(long long)plan_block() * kNQ + 0] = t[0];
        part[(long long)plan_block() * kNQ + 1] = t[1];
    }
}

void launch_cg_update(hipStream_t s, const Plan &p, const Rep *rep, RepState *st, Chain ch, int init,
                      double *w, double *g, const double *gt, double *d, const double *phit, double *part)
{
    hipLaunchKernelGGL(k_cg_update, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, st, ch.nsp,
                       ch.precond, p.span, init, w, g, gt, d, phit, part);
}

// Solvent density of eq. 2, phi_S = phibar_s exp(-w_S) / <exp(-w_S)>, into the field-layout
// output (after the sweeps whose density launch does not write it itself).
__global__ __launch_bounds__(kBlock) void k_solvent(const int *__restrict__ blk_rep,
                                                    const int *__restrict__ blk_first,
                                                    const Rep *__restrict__ rep, const RepState *__restrict__ st,
                                                    int nsp, const double *__restrict__ w, double *__restrict__ out)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    const long long k = off_field(R, nsp) + 2 * V + i;
    const RepState &S = st[sr.r];
    out[k] = S.phibar_s * exp(-w[k]) / S.sol_mean;
}

void launch_solvent(hipStream_t s, const Plan &p, const Rep *rep, RepState *st, Chain ch, const double *w,
                    double *out)
{
    hipLaunchKernelGGL(k_solvent, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, st, ch.nsp, w,
                       out);
}

}  // namespace hsf
