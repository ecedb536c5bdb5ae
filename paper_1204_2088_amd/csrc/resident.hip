// resident.hip -- evaluations and inversions of boxes of at most 16^3 in one workgroup per
// replica.
//
// A 16^3 box has 16 workgroups' worth of sites per contour step: the sweeps are chains of
// launches of 4 us each whatever the box holds, a pass of the inversion 12 of them (51 us)
// and the host's turn between passes another 13 us.  Here one workgroup of 1024 threads holds the
// propagator of a replica in LDS and the field factors in registers and runs whole
// evaluations, and with them whole inversions (the line searches' scalar logic included), in
// one launch.  A thread owns four planes of one column (x, y).  The LDS layout is fixed at
// 16 x 16 sites a plane with one halo plane at each end, so the 54 reads of a thread's four
// stencils are nine registers with constant offsets and no address arithmetic (consecutive
// lanes read consecutive sites: no bank conflicts); with the box's own strides the
// addresses cost more instructions than the sums.  Only G_s goes to memory and comes back to
// the same thread; the density sums stay in registers.
//
// Bound by the instructions of one CU (a replica has no more): an evaluation of 16^3 A4B4 in
// FP64 takes 35.8 us (80 with the box's strides, 61 before the x neighbours and the wavefront
// sums moved from LDS to DPP, 39 with both rows' x neighbours summed), an hsf_evaluate call 52
// us against 90 by launches, a coupled step 1.61 ms against 3.3.  Up to 256 replicas, one per CU, the chain of launches is
// never faster: 4^3 45 us against 68, 16^3 46 against 68 (one replica, FP32); 512 of 16^3 115
// against 378.  With more, boxes of at most 64 sites leave too many threads idle (1024 of 8^3 169 us
// against 214, 1024 of 4^3 with 8 beads 167 against 174, with 64 beads 782 against 729, 4096 of 4^3 606 against
// 536), so hsf_autotune times both.  Larger boxes do not fit: 32^3 would need 8 times the LDS.
//
// Every stored value is the same expression of the same operands as in the one-step
// kernels (in FP64 with 16-site rows up to the order of the four corner neighbours); sums over
// sites have their own fixed order.
#include <algorithm>

#include "ctl_device.h"
#include "resident.h"

namespace hsf {

constexpr int kResThreads = 1024, kResWaves = kResThreads / 64;
constexpr int kResSums = 70;   // per-wavefront partial sums: N + 2 steps' or a phase's slots

struct ResShared {
    RepState S;
    Chain ch;
    double ws[kResWaves][kResSums];
    double vals[kResSums];
};

// x neighbours in rows of 16 lanes taken as rings (row_ror:1 and row_ror:15), summed.
__device__ __forceinline__ float row_sums(float v)
{
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(b, 0x121, 0xf, 0xf, true)) +
           __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(b, 0x12f, 0xf, 0xf, true));
}
__device__ __forceinline__ double row_sums(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int l0 = __builtin_amdgcn_mov_dpp((int)b, 0x121, 0xf, 0xf, true);
    const int l1 = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x121, 0xf, 0xf, true);
    const int r0 = __builtin_amdgcn_mov_dpp((int)b, 0x12f, 0xf, 0xf, true);
    const int r1 = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x12f, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)l1 << 32) | (unsigned int)l0) +
           __builtin_bit_cast(double, ((long long)r1 << 32) | (unsigned int)r0);
}

// Sums over the workgroup of NV values per thread into sh.vals[0 .. NV - 1] (fixed order).
template <int NV>
__device__ __forceinline__ void res_reduce(ResShared &sh, double (&v)[NV])
{
    const int lane = (int)threadIdx.x & 63, wid = (int)threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        v[q] = wave_sum(v[q]);
        if (lane == 0) sh.ws[wid][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double t = 0.0;
        for (int k = 0; k < kResWaves; ++k) t += sh.ws[k][threadIdx.x];
        sh.vals[threadIdx.x] = t;
    }
    __syncthreads();
}

// A phase's scalar logic (one thread), between barriers.
__device__ __forceinline__ void res_control(ResShared &sh, int phase, const Chain &ch, const Rep &R, const double *gsum,
                                            double tol, int max_iter)
{
    if (threadIdx.x == 0) control(sh.S, phase, ch, sh.vals, gsum, (double)R.V, R.csum, tol, max_iter);
    __syncthreads();
}

// Planes of the LDS layout: site (x, y, z) at x + 16 y + 256 (z + 1), halo planes 0 and Lz + 1.
constexpr int kResEdge = 16, kResArea = kResEdge * kResEdge, kResSlots = kResArea * (kResEdge + 2);

// The column of a thread: sites (x, y, z0 + j), j < n (uniform).  Threads outside the box's
// rows (live not set) compute on the layout's unused sites and store nothing to memory.
struct ResCol {
    int n, z0;
    bool live;
    int area;            // sites of a plane of the box
    unsigned gb;         // x + Lx y in the arrays of the box
    int o[9];            // in-plane LDS offsets: rows y, y - 1, y + 1; x - 1, x, x + 1 of each

    __device__ __forceinline__ void init(const Rep &R)
    {
        const int c = (int)threadIdx.x & (kResArea - 1), x = c & (kResEdge - 1), y = c / kResEdge;
        area = R.Lx * R.Ly;
        z0 = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kResArea) * kResZ;
        n = max(0, min(kResZ, R.Lz - z0));
        live = x < R.Lx && y < R.Ly && n > 0;
        gb = (unsigned)(x + R.Lx * y);
        const int xs[3] = {wrap1(x - 1, R.Lx), x, wrap1(x + 1, R.Lx)};
        const int ys[3] = {y, wrap1(y - 1, R.Ly), wrap1(y + 1, R.Ly)};
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int b = 0; b < 3; ++b)
                o[3 * a + b] = x < R.Lx && y < R.Ly ? ys[a] * kResEdge + xs[b] : y * kResEdge + x;
    }
    // element j of the column in an array of the box (uniform base, the lane's offset)
    template <typename T>
    __device__ __forceinline__ T &at(T *f, int j) const
    {
        return *(T *)((char *)(f + (long long)(z0 + j) * area) + gb * (unsigned)sizeof(T));
    }
    // The compiler would keep every address derived from the column in registers over the
    // steps and passes and spill; after this it forms them anew.
    __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(gb)); }
};

// The column's value j into the LDS propagator f, and into the halo plane it is the image of.
template <typename real>
__device__ __forceinline__ void res_put(real *f, const ResCol &c, int Lz, int j, real v)
{
    const int z = c.z0 + j;   // uniform
    if (z >= Lz) return;
    f[c.o[1] + (z + 1) * kResArea] = v;
    if (z == 0) f[c.o[1] + (Lz + 1) * kResArea] = v;
    if (z == Lz - 1) f[c.o[1]] = v;
}

// The stencil of f on the column's planes (the sums of column_stencil).  X16: rows of
// exactly 16 sites, whose x neighbours are the adjacent lanes of a row of 16: 18 reads instead
// of 54.  There the corner sum of FP64 takes the x neighbours of the two rows' sum, which is a
// sixth of a step's instructions less than the sum of both rows' neighbours.
template <typename real, bool X16>
__device__ __forceinline__ void res_stencil(const real *f, const ResCol &c, real c0, real c1, real c2, real c3,
                                            real (&S)[kResZ])
{
    const real *p = f + c.z0 * kResArea;
    const int *o = c.o;
    real a0[kResZ + 2], a1[kResZ + 2], a2[kResZ + 2];
#pragma unroll
    for (int q = 0; q < kResZ + 2; ++q) {
        const int k = q * kResArea;
        if constexpr (X16) {
            const real v = p[o[1] + k], m = p[o[4] + k], n = p[o[7] + k];
            const real mn = m + n;
            a0[q] = v;
            a1[q] = row_sums(v) + mn;
            if constexpr (sizeof(real) == 8) a2[q] = row_sums(mn);
            else a2[q] = row_sums(m) + row_sums(n);   // the one-step kernels' order, bit for bit
        } else {
            a0[q] = p[o[1] + k];
            a1[q] = (p[o[0] + k] + p[o[2] + k]) + (p[o[4] + k] + p[o[7] + k]);
            a2[q] = (p[o[3] + k] + p[o[5] + k]) + (p[o[6] + k] + p[o[8] + k]);
        }
    }
#pragma unroll
    for (int j = 0; j < kResZ; ++j)
        S[j] = c0 * a0[j + 1] + c1 * (a1[j + 1] + (a0[j] + a0[j + 2])) + c2 * (a2[j + 1] + (a1[j] + a1[j + 2])) +
               c3 * (a2[j] + a2[j + 2]);
}

// One density-functional evaluation of the replica: its polymer density sums (before the
// normalisation by coef) in a[plane][species], Q in the state; with `sums` also the sums of
// every step's G_s and of E_A, E_B in vals[0 .. N + 1].
template <typename real, bool X16>
__device__ __forceinline__ void res_evaluate(ResShared &sh, real *lds, ResCol &c, const Rep &R, const Chain &ch,
                                             real *__restrict__ G, const double *__restrict__ w,
                                             const double *__restrict__ d, bool use_alpha, bool sums,
                                             double (&a)[kResZ][2])
{
    const int V = (int)R.V, N = ch.N, Lz = R.Lz;
    real *g0 = lds, *g1 = lds + kResSlots;
    const real c0 = (real)R.c[0], c1 = (real)R.c[1], c2 = (real)R.c[2], c3 = (real)R.c[3], csum = (real)R.csum;
    const int lane = (int)threadIdx.x & 63, wid = (int)threadIdx.x >> 6;
    const double alpha = use_alpha ? sh.S.alpha : 0.0;
    real E[kResZ][2];
    auto row_sum = [&](double v, int row) {
        v = wave_sum(v);
        if (lane == 0) sh.ws[wid][row] = v;
    };
    // field factors, and G_1 (a column's planes past its last and dead lanes: factor 0, no sums)
    {
        const real sc = (real)ldexp(1.0, -sh.S.scale_e[0]);
        const int t1 = ch.types[0];
        double es[2] = {0.0, 0.0}, gs = 0.0;
#pragma unroll
        for (int j = 0; j < kResZ; ++j) {
            E[j][0] = E[j][1] = (real)0;
            if (j < c.n && c.live) {
#pragma unroll
                for (int I = 0; I < 2; ++I) {
                    double x = c.at(w + I * V, j);
                    if (use_alpha) x = fma(alpha, c.at(d + I * V, j), x);
                    E[j][I] = (real)exp(-x);
                    es[I] += (double)E[j][I];
                }
            }
            const real g = (t1 ? E[j][1] : E[j][0]) * csum * sc;
            res_put(g0, c, Lz, j, g);
            if (j < c.n && c.live) c.at(G, j) = g;
            gs += (double)g;
        }
        if (sums || N == 1) row_sum(gs, 0);
        if (sums) {
            row_sum(es[0], N);
            row_sum(es[1], N + 1);
        }
    }
    __syncthreads();
    for (int s = 2; s <= N; ++s) {
        c.fresh();
        const real sc = (real)ldexp(1.0, -sh.S.scale_e[s - 1]);
        const int ts = ch.types[s - 1];
        real *Gs = G + (long long)(s - 1) * V;
        real S[kResZ];
        res_stencil<real, X16>(g0, c, c0, c1, c2, c3, S);
#pragma unroll
        for (int j = 0; j < kResZ; ++j) {
            S[j] = (ts ? E[j][1] : E[j][0]) * S[j] * sc;
            res_put(g1, c, Lz, j, S[j]);
        }
        if (c.live) {
#pragma unroll
            for (int j = 0; j < kResZ; ++j)
                if (j < c.n) c.at(Gs, j) = S[j];
        }
        if (sums || s == N) {   // planes and lanes outside the box hold 0
            double gs = 0.0;
#pragma unroll
            for (int j = 0; j < kResZ; ++j) gs += (double)S[j];
            row_sum(gs, s - 1);
        }
        __syncthreads();
        real *t = g0;
        g0 = g1;
        g1 = t;
    }
    // the sums over the wavefronts: G_N's (Q) and, with `sums`, every row
    if ((int)threadIdx.x <= N + 1 && (sums || (int)threadIdx.x == N - 1)) {
        double t = 0.0;
        for (int k = 0; k < kResWaves; ++k) t += sh.ws[k][threadIdx.x];
        sh.vals[threadIdx.x] = t;
    }
    // G+_N and bead N's term, then the backward steps; a term is rounded to the propagators'
    // precision, bead 1's product is kept in FP64
    {
        const real sc = (real)ldexp(1.0, -sh.S.scale_e[N - 1]);
        const int ts = ch.types[N - 1];
#pragma unroll
        for (int j = 0; j < kResZ; ++j) {
            a[j][0] = a[j][1] = 0.0;
            const real gv = j < c.n ? g0[c.o[1] + (c.z0 + j + 1) * kResArea] : (real)0;
            const double term = N == 1 ? (double)gv * (double)csum : (double)(real)(gv * csum);
            if (ts == 0) a[j][0] += term;
            else a[j][1] += term;
            res_put(g1, c, Lz, j, (ts ? E[j][1] : E[j][0]) * csum * sc);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        bool bad;
        q_from_sum(sh.vals[N - 1], (double)R.V, sh.S.scale_e, N, sh.S.q, sh.S.ln_q, bad);
        if (bad) sh.S.nonfinite = 1;
    }
    if (N == 1) __syncthreads();   // Q for every wavefront; longer chains have the barriers below
    real *gp = g1, *gn = g0;
    for (int s = N - 1; s >= 1; --s) {
        c.fresh();
        const real sc = (real)ldexp(1.0, -sh.S.scale_e[s - 1]);
        const int ts = ch.types[s - 1];
        real *Gs = G + (long long)(s - 1) * V;
        real S[kResZ], gv[kResZ];
#pragma unroll
        for (int j = 0; j < kResZ; ++j) gv[j] = (real)0;
        if (c.live) {
#pragma unroll
            for (int j = 0; j < kResZ; ++j)
                if (j < c.n) gv[j] = c.at(Gs, j);
        }
        res_stencil<real, X16>(gp, c, c0, c1, c2, c3, S);
        if (s > 1) {
#pragma unroll
            for (int j = 0; j < kResZ; ++j) res_put(gn, c, Lz, j, (ts ? E[j][1] : E[j][0]) * S[j] * sc);
        }
        double term[kResZ];
#pragma unroll
        for (int j = 0; j < kResZ; ++j)
            term[j] = s == 1 ? (double)gv[j] * (double)S[j] : (double)(real)(gv[j] * S[j]);
        if (ts == 0) {
#pragma unroll
            for (int j = 0; j < kResZ; ++j) a[j][0] += term[j];
        } else {
#pragma unroll
            for (int j = 0; j < kResZ; ++j) a[j][1] += term[j];
        }
        __syncthreads();
        real *t = gp;
        gp = gn;
        gn = t;
    }
}

// kind RES_EVAL: hsf_evaluate's sequence, densities into out (field layout).  RES_START: the
// start of an inversion, then passes; RES_PASSES: further passes.  At most max_passes passes
// per launch (the host launches again while a replica is active).
template <typename real, bool X16>
__global__ __launch_bounds__(kResThreads) void k_resident(int kind, const Rep *__restrict__ rep,
                                                          RepState *__restrict__ st, Chain chain,
                                                          real *__restrict__ Gall,
                                                          double *__restrict__ wall, double *__restrict__ dall,
                                                          const double *__restrict__ phiall,
                                                          double *__restrict__ outall, double tol, int max_iter,
                                                          int max_passes, RepState *__restrict__ mirror)
{
    extern __shared__ __align__(16) unsigned char smem[];
    ResShared &sh = *reinterpret_cast<ResShared *>(smem);
    real *lds = reinterpret_cast<real *>(smem + ((sizeof(ResShared) + 15) & ~(size_t)15));
    const int r = (int)blockIdx.x;
    const Rep R = rep[r];
    const int V = (int)R.V;
    {
        const int *src = reinterpret_cast<const int *>(&st[r]);
        int *dst = reinterpret_cast<int *>(&sh.S);
        for (int k = (int)threadIdx.x; k < (int)(sizeof(RepState) / 4); k += kResThreads) dst[k] = src[k];
        if (threadIdx.x == 0) sh.ch = chain;
        // sites of the layout outside the box are read with factor 0: finite values
        for (int k = (int)threadIdx.x; k < 2 * kResSlots; k += kResThreads) lds[k] = (real)0;
    }
    __syncthreads();
    const Chain &ch = sh.ch;
    if (kind == RES_PASSES && !sh.S.active) return;   // finished (uniform)
    ResCol c;
    c.init(R);
    real *G = Gall + (long long)ch.N * R.site_off;
    double *w = wall + off_field(R, ch.nsp), *d = dall + off_poly(R);
    const double *phi = phiall + off_field(R, ch.nsp);
    double a[kResZ][2];

    if (kind != RES_PASSES) {
        // target amounts and norms, means of the fields, <exp(-w_S)>
        double v[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < kResZ; ++j) {
                if (j >= c.n || !c.live) continue;
                const double pa = c.at(phi, j), pb = c.at(phi + V, j);
                v[0] += pa + pb;
                if (ch.nsp == 3) {
                    v[1] += c.at(phi + 2 * V, j);
                    if (kind == RES_EVAL) v[6] += exp(-c.at(w + 2 * V, j));
                }
                v[2] += pa * pa;
                v[3] += pb * pb;
                v[4] += c.at(w, j);
                v[5] += c.at(w + V, j);
            }
        res_reduce(sh, v);
        res_control(sh, kind == RES_EVAL && ch.nsp == 3 ? PH_TARGET_SOLVENT : PH_TARGET, ch, R, nullptr, tol, max_iter);
    }
    if (kind == RES_START) {
        // gauge and closed-form solvent field
#pragma unroll
            for (int j = 0; j < kResZ; ++j) {
                if (j >= c.n || !c.live) continue;
                c.at(w, j) -= sh.S.wmean[0];
                c.at(w + V, j) -= sh.S.wmean[1];
                if (ch.nsp == 3) c.at(w + 2 * V, j) = -log(c.at(phi + 2 * V, j) / sh.S.phibar_s);
            }
    }
    for (int pass = 0;; ++pass) {
        const bool first = kind != RES_PASSES && pass == 0;
        c.fresh();
        __syncthreads();
        res_evaluate<real, X16>(sh, lds, c, R, ch, G, w, d, !first, first, a);
        c.fresh();
        const double coef = sh.S.phibar_p / ((double)ch.N * sh.S.q);
        if (kind == RES_EVAL) {
            double *out = outall + off_field(R, ch.nsp);
#pragma unroll
                for (int j = 0; j < kResZ; ++j) {
                    if (j >= c.n || !c.live) continue;
                    c.at(out, j) = coef * a[j][0];
                    c.at(out + V, j) = coef * a[j][1];
                    if (ch.nsp == 3) c.at(out + 2 * V, j) = sh.S.phibar_s * exp(-c.at(w + 2 * V, j)) / sh.S.sol_mean;
                }
            __syncthreads();
            res_control(sh, PH_SCALES, ch, R, sh.vals, tol, max_iter);
            break;
        }
        // the gradient phi^t - phi (in place of the density sums) and its dot products d.g,
        // g.z, |g_A|^2, |g_B|^2; the sums of the steps move behind those four slots
        double t[4] = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < kResZ; ++j) {
                if (j >= c.n || !c.live) continue;
#pragma unroll
                for (int I = 0; I < 2; ++I) {
                    const double pt = c.at(phi + I * V, j), gI = pt - coef * a[j][I];
                    a[j][I] = gI;
                    if (!first) t[0] += c.at(d + I * V, j) * gI;
                    t[1] += ch.precond ? gI * gI / pt : gI * gI;
                    t[2 + I] += gI * gI;
                }
            }
        double keep = 0.0;
        if ((int)threadIdx.x < ch.N + 2) keep = sh.vals[threadIdx.x];
        __syncthreads();
        res_reduce(sh, t);
        if (first && (int)threadIdx.x < ch.N + 2) sh.vals[4 + threadIdx.x] = keep;
        __syncthreads();
        res_control(sh, first ? PH_EVAL0 : PH_TRIAL, ch, R, sh.vals + 4, tol, max_iter);
        const bool pending = sh.S.pending != 0;
        if (first ? pending : sh.S.accepted != 0) {
            // the conjugate-gradient update, d.g and d H d, and the start of the next line search
            const double alpha = sh.S.alpha, beta = sh.S.beta;
            const bool upd_d = first || !sh.S.done;
            double u[2] = {0, 0};
            c.fresh();
#pragma unroll
                for (int j = 0; j < kResZ; ++j) {
                    if (j >= c.n || !c.live) continue;
#pragma unroll
                    for (int I = 0; I < 2; ++I) {
                        const double gI = a[j][I], pt = c.at(phi + I * V, j);
                        double dI = first ? 0.0 : c.at(d + I * V, j);
                        if (!first) c.at(w + I * V, j) = fma(alpha, dI, c.at(w + I * V, j));
                        if (upd_d) {
                            const double z = ch.precond ? gI / pt : gI;
                            dI = first ? -z : fma(beta, dI, -z);
                            c.at(d + I * V, j) = dI;
                        }
                        u[0] += dI * gI;
                        u[1] += dI * dI * pt;
                    }
                }
            __syncthreads();
            res_reduce(sh, u);
            if (pending) {
                res_control(sh, PH_BEGIN, ch, R, nullptr, tol, max_iter);
            } else {
                if (threadIdx.x == 0) sh.S.accepted = 0;
                __syncthreads();
            }
        }
        if (!sh.S.active || pass + 1 >= max_passes) break;
    }
    __syncthreads();
    {
        const int *src = reinterpret_cast<const int *>(&sh.S);
        int *dst = reinterpret_cast<int *>(&st[r]), *hm = reinterpret_cast<int *>(&mirror[r]);
        for (int k = (int)threadIdx.x; k < (int)(sizeof(RepState) / 4); k += kResThreads) {
            dst[k] = src[k];
            hm[k] = src[k];
        }
    }
}

namespace {

size_t res_lds(size_t rs) { return ((sizeof(ResShared) + 15) & ~(size_t)15) + 2 * (size_t)kResSlots * rs; }

}  // namespace

bool resident_fits(const Rep *reps, int n_rep, size_t real_bytes, size_t lds_limit)
{
    for (int r = 0; r < n_rep; ++r)
        if (reps[r].Lx > kResEdge || reps[r].Ly > kResEdge || reps[r].Lz > kResEdge) return false;
    return res_lds(real_bytes) <= lds_limit;
}

template <typename real>
hipError_t launch_resident(hipStream_t s, int kind, const Rep *reps_host, int n_rep, const Rep *rep, RepState *st,
                           const Chain &ch, real *G, double *w, double *d, const double *phi, double *out, double tol,
                           int max_iter, int max_passes, RepState *mirror)
{
    const size_t lds = res_lds(sizeof(real));
    bool x16 = true;
    for (int r = 0; r < n_rep; ++r) x16 = x16 && reps_host[r].Lx == kResEdge;
    auto kern = x16 ? k_resident<real, true> : k_resident<real, false>;
    // more than the default 64 KB of LDS per workgroup
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(n_rep), dim3(kResThreads), lds, s, kind, rep, st, ch, G, w, d, phi, out, tol,
                       max_iter, max_passes, mirror);
    return hipGetLastError();
}

template hipError_t launch_resident<float>(hipStream_t, int, const Rep *, int, const Rep *, RepState *, const Chain &,
                                           float *, double *, double *, const double *, double *, double, int, int,
                                           RepState *);
template hipError_t launch_resident<double>(hipStream_t, int, const Rep *, int, const Rep *, RepState *, const Chain &,
                                            double *, double *, double *, const double *, double *, double, int, int,
                                            RepState *);

}  // namespace hsf
