// dyn.hip -- the dynamics around the density functional:
//   chemical potential (eq. 4) and thermodynamic force (eq. 8);
//   D3Q19 lattice Boltzmann, moments (eq. 9), equilibrium (eq. 11), single-relaxation
//   collision L_ij = -delta_ij / tau with its forcing term, collide then stream (eq. 10);
//   conservative convection-diffusion update (eq. 3);
//   optional thermal noise: LB mode noise (eq. 13) and composition noise (eq. 5).
#include <hip/hip_ext.h>
#include <math.h>

#include <type_traits>

#include "device_common.h"
#include "philox.h"

namespace hsf {

// D3Q19 velocities: rest, 6 faces, 12 edges (order documented in hsf.h).
constexpr int kCx[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
constexpr int kCy[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
constexpr int kCz[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};

// Weights of eq. 11.
__host__ __device__ constexpr double lb_w(int q) { return q == 0 ? 1.0 / 3.0 : (q < 7 ? 1.0 / 18.0 : 1.0 / 36.0); }

// LB populations in memory: FP64 values n_i, or (FP32 storage) the deviations n_i - w_i
// from the rest state, whose magnitude is that of the flow and density perturbations, so
// FP32 keeps about 7 significant digits of the perturbation rather than of n_i.  All
// arithmetic is FP64.
__device__ __forceinline__ double pop_load(const double *p, long long k, int) { return p[k]; }
__device__ __forceinline__ double pop_load(const float *p, long long k, int q) { return lb_w(q) + (double)p[k]; }
__device__ __forceinline__ void pop_store(double *p, long long k, int, double v) { p[k] = v; }
__device__ __forceinline__ void pop_store(float *p, long long k, int q, double v) { p[k] = (float)(v - lb_w(q)); }

__device__ __forceinline__ void site_xyz(const Rep &R, long long i, int &x, int &y, int &z)
{
    x = (int)(i % R.Lx);
    y = (int)((i / R.Lx) % R.Ly);
    z = (int)(i / ((long long)R.Lx * R.Ly));
}

__device__ __forceinline__ long long sidx(const Rep &R, int x, int y, int z)
{
    return (long long)x + (long long)R.Lx * ((long long)y + (long long)R.Ly * z);
}

// A wavefront's part of the column plan: P consecutive x sites per lane of one row, CZ core
// planes.  Rows of exactly 64 P sites are whole (the lanes form the periodic ring); others
// are cut into pieces with a halo site at both ends, whose lanes compute and store nothing.
// SHORT: rows of at most 30 sites stand side by side in the wavefront, each with its two halo
// sites (row and the y neighbours are then the lane's own).  Every lane's address is inside the box.
template <int P, int CZ, bool SHORT>
struct Col {
    int r, y, z0, nz, plane, Lz;
    long long V, row, up, dn;    // offsets of the row and of its y neighbours within a plane
    unsigned xb;                 // the lane's byte offset in a row
    bool core;                   // its sites are the wavefront's to store

    __device__ __forceinline__ bool init(const int *blk_rep, const int *blk_first, const Rep *rep)
    {
        const int pb = plan_block();
        r = blk_rep[pb];
        const Rep &R = rep[r];
        const RowsCut cut = rows_cut(R.Lx, P, 1);
        int lb = pb - blk_first[r];
        const int x0 = (lb % cut.ntx) * cut.width;
        lb /= cut.ntx;
        const int rows = SHORT ? col_rows(0, R.Lx) : 1, nty = (R.Ly + kColY * rows - 1) / (kColY * rows);
        y = ((lb % nty) * kColY + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) * rows;
        z0 = (lb / nty) * CZ;
        if (y >= R.Ly) return false;
        int lane = (int)threadIdx.x & 63;
        bool mine = true;
        if (SHORT && rows > 1) {
            const int k = lane / (R.Lx + 2);
            lane -= k * (R.Lx + 2);
            mine = k < rows && y + k < R.Ly;
            y = min(y + k, R.Ly - 1);
        }
        Lz = R.Lz;
        nz = min(CZ, Lz - z0);
        V = R.V;
        plane = R.Lx * R.Ly;
        row = (long long)y * R.Lx;
        dn = (long long)wrap1(y - 1, R.Ly) * R.Lx;
        up = (long long)wrap1(y + 1, R.Ly) * R.Lx;
        const int xu = x0 - cut.halo + lane * P;
        core = mine && xu >= x0 && xu < x0 + cut.width && xu < R.Lx;
        int x = xu % R.Lx;
        if (x < 0) x += R.Lx;
        xb = (unsigned)x * (unsigned)sizeof(double);
        return true;
    }
    // offset of plane z0 - 1 + q, q = 0 .. CZ + 1 (past a short last chunk: its end)
    __device__ __forceinline__ long long z(int q) const
    {
        return (long long)wrap1(min(z0 - 1 + q, z0 + nz), Lz) * plane;
    }
    __device__ __forceinline__ Sites<double, P> load(const double *f, long long off) const
    {
        Sites<double, P> v;
        __builtin_memcpy(&v, reinterpret_cast<const char *>(f + off) + xb, sizeof v);
        return v;
    }
    __device__ __forceinline__ void store(double *f, long long off, const Sites<double, P> &v) const
    {
        __builtin_memcpy(reinterpret_cast<char *>(f + off) + xb, &v, sizeof v);
    }
};

template <int P>
__device__ __forceinline__ void x_pair(const Sites<double, P> &c, Sites<double, P> &l, Sites<double, P> &h)
{
    if constexpr (P == 1) {
        l.s[0] = ring_left(c.s[0]);
        h.s[0] = ring_right(c.s[0]);
    } else {
        l = {{ring_left(c.s[1]), c.s[0]}};
        h = {{c.s[1], ring_right(c.s[0])}};
    }
}

// mu_I = -w_I + sum_J chi_IJ sigma[phi_J] + kappa (sum_J phi_J - 1).  One species at a time,
// each wavefront loads the three rows around its own on kMuZ + 2 planes (3 (kMuZ + 2) /
// kMuZ = 4.5 loads per site, x neighbours from the adjacent lanes) and combines three
// planes' class sums per site.  With one site per lane and its nine rows loaded anew (18
// loads per site and species) the kernel was bound by its loads' latency: 85 us for 3 species
// at 128^3 (151 MB); now 36 us, 4.2 TB/s.  A box of 4 x 256 x 256 leaves most lanes idle with a
// wavefront per row: potential and force 45 us a call, 27 with one site per lane of the whole box, 15
// with ten rows side by side.
template <int NSP, int P, bool SHORT>
__global__ __launch_bounds__(kBlock) void k_mu(const int *__restrict__ blk_rep, const int *__restrict__ blk_first,
                                               const Rep *__restrict__ rep, const double *__restrict__ phi,
                                               const double *__restrict__ w, double *__restrict__ mu)
{
    typedef Sites<double, P> row_t;
    constexpr int CZ = kMuZ;
    Col<P, CZ, SHORT> t;
    if (!t.init(blk_rep, blk_first, rep)) return;
    const Rep &R = rep[t.r];
    const long long fo = off_field(R, NSP);
    const double c0 = R.c[0], c1 = R.c[1], c2 = R.c[2], c3 = R.c[3];
    row_t inter[NSP][CZ], tot[CZ];
#pragma unroll
    for (int j = 0; j < CZ; ++j)
#pragma unroll
        for (int u = 0; u < P; ++u) {
            tot[j].s[u] = 0.0;
#pragma unroll
            for (int I = 0; I < NSP; ++I) inter[I][j].s[u] = 0.0;
        }
#pragma unroll 1
    for (int J = 0; J < NSP; ++J) {
        const double *f = phi + fo + (long long)J * t.V;
        row_t c[CZ + 2], m[CZ + 2], p[CZ + 2];
#pragma unroll
        for (int q = 0; q < CZ + 2; ++q) {
            const long long zq = t.z(q);
            c[q] = t.load(f, zq + t.row);
            m[q] = t.load(f, zq + t.dn);
            p[q] = t.load(f, zq + t.up);
        }
        row_t a1[CZ + 2], a2[CZ + 2];
#pragma unroll
        for (int q = 0; q < CZ + 2; ++q) {
            const row_t ec = x_sums(c[q]), em = x_sums(m[q]), ep = x_sums(p[q]);
#pragma unroll
            for (int u = 0; u < P; ++u) {
                a1[q].s[u] = ec.s[u] + (m[q].s[u] + p[q].s[u]);
                a2[q].s[u] = em.s[u] + ep.s[u];
            }
        }
#pragma unroll
        for (int j = 0; j < CZ; ++j)
#pragma unroll
            for (int u = 0; u < P; ++u) {
                const double sp = c0 * c[j + 1].s[u] + c1 * (a1[j + 1].s[u] + (c[j].s[u] + c[j + 2].s[u])) +
                                  c2 * (a2[j + 1].s[u] + (a1[j].s[u] + a1[j + 2].s[u])) +
                                  c3 * (a2[j].s[u] + a2[j + 2].s[u]);
                tot[j].s[u] += c[j + 1].s[u];
#pragma unroll
                for (int I = 0; I < NSP; ++I) inter[I][j].s[u] += R.chi[I][J] * sp;
            }
    }
    if (!t.core) return;
#pragma unroll
    for (int j = 0; j < CZ; ++j) {
        if (j >= t.nz) continue;
        const long long o = (long long)(t.z0 + j) * t.plane + t.row;
#pragma unroll
        for (int I = 0; I < NSP; ++I) {
            const long long k = fo + (long long)I * t.V + o;
            const row_t wv = t.load(w, k);
            row_t v;
#pragma unroll
            for (int u = 0; u < P; ++u) v.s[u] = -wv.s[u] + inter[I][j].s[u] + R.kappa * (tot[j].s[u] - 1.0);
            t.store(mu, k, v);
        }
    }
}

// f = -dt^2 sum_I phi_I (mu_I(r + e) - mu_I(r - e)) / 2 per axis (LB units).
__global__ __launch_bounds__(kBlock) void k_force(const int *__restrict__ blk_rep,
                                                  const int *__restrict__ blk_first, const Rep *__restrict__ rep,
                                                  Chain ch, const double *__restrict__ phi,
                                                  const double *__restrict__ mu, double *__restrict__ f)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    int x, y, z;
    site_xyz(R, i, x, y, z);
    const long long fo = off_field(R, ch.nsp);
    const long long nb[6] = {sidx(R, wrap1(x + 1, R.Lx), y, z), sidx(R, wrap1(x - 1, R.Lx), y, z),
                             sidx(R, x, wrap1(y + 1, R.Ly), z), sidx(R, x, wrap1(y - 1, R.Ly), z),
                             sidx(R, x, y, wrap1(z + 1, R.Lz)), sidx(R, x, y, wrap1(z - 1, R.Lz))};
    double acc[3] = {0, 0, 0};
    for (int I = 0; I < ch.nsp; ++I) {
        const double *m = mu + fo + I * V;
        const double p = phi[fo + I * V + i];
#pragma unroll
        for (int a = 0; a < 3; ++a) acc[a] += p * (0.5 * (m[nb[2 * a]] - m[nb[2 * a + 1]]));
    }
    const double k = -R.dt * R.dt;
    const long long vo = 3LL * R.site_off;
#pragma unroll
    for (int a = 0; a < 3; ++a) f[vo + a * V + i] = k * acc[a];
}

// Multiple-relaxation-time collision (eq. 12-14) in the orthogonal basis of Table 1:
// e_k(c) for k = 0..18, orthogonal under the weights w_i; b_k = sum_i w_i e_k(c_i)^2.
__host__ __device__ constexpr double mrt_e(int k, int cx, int cy, int cz)
{
    const double x = cx, y = cy, z = cz, c2 = x * x + y * y + z * z;
    switch (k) {
    case 0: return 1.0;
    case 1: return x;
    case 2: return y;
    case 3: return z;
    case 4: return c2 - 1.0;
    case 5: return x * x - y * y;
    case 6: return c2 - 3.0 * z * z;
    case 7: return x * y;
    case 8: return x * z;
    case 9: return y * z;
    case 10: return (3.0 * c2 - 5.0) * x;
    case 11: return (3.0 * c2 - 5.0) * y;
    case 12: return (3.0 * c2 - 5.0) * z;
    case 13: return (y * y - z * z) * x;
    case 14: return (z * z - x * x) * y;
    case 15: return (x * x - y * y) * z;
    case 16: return 3.0 * c2 * c2 - 6.0 * c2 + 1.0;
    case 17: return (2.0 * c2 - 3.0) * (x * x - y * y);
    default: return (2.0 * c2 - 3.0) * (c2 - 3.0 * z * z);
    }
}


// The basis at the 19 velocities, 1 / b_k and its square root, as compile-time tables (the
// unrolled projections below index them with constants).
struct MrtTable {
    double e[19][19];   // [k][q]
    double binv[19], rbinv[19];
};

constexpr MrtTable make_mrt_table()
{
    MrtTable t{};
    for (int k = 0; k < 19; ++k) {
        double b = 0.0;
        for (int q = 0; q < 19; ++q) {
            t.e[k][q] = mrt_e(k, kCx[q], kCy[q], kCz[q]);
            b += lb_w(q) * t.e[k][q] * t.e[k][q];
        }
        t.binv[k] = 1.0 / b;
        double r = 1.0;
        for (int it = 0; it < 60; ++it) r = 0.5 * (r + t.binv[k] / r);
        t.rbinv[k] = r;
    }
    return t;
}

__device__ constexpr MrtTable kMrt = make_mrt_table();

// Velocities 2 p + 1 and 2 p + 2 are opposite: modes even in c see the sum of a pair, odd ones the
// difference, so a transform takes half the terms, and those with e_k = 0 are left out (the
// compiler has to keep a product with zero): about 100 terms where 19 x 19 are written out.
constexpr bool mrt_odd(int k) { return (k >= 1 && k <= 3) || (k >= 10 && k <= 15); }

// sum_k e_k(c) v_k over the even (odd) modes K0 .. 18 at velocity q.
template <int K0, bool ODD>
__device__ __forceinline__ double mrt_back(const double *v, int q)
{
    double a = 0.0;
    bool first = true;
#pragma unroll
    for (int k = K0; k < 19; ++k) {
        const double e = kMrt.e[k][q];
        if (mrt_odd(k) != ODD || e == 0.0) continue;
        a = first ? e * v[k] : a + e * v[k];
        first = false;
    }
    return a;
}

// Collision of one site by the MRT scheme: n* = n_eq + w_i sum_k e_k(c_i) m*_k / b_k with m*_k =
// gamma_k (n - n_eq)_k + (Delta^f)_k, where the forcing Delta^f_i = (w_i / c_s^2) [f.c_i + Sigma :
// (c_i c_i - c_s^2 1) / (2 c_s^2)] and Sigma = (1 + gamma_s)/2 (u f + f u - 2/3 (u.f) 1) + (1 +
// gamma_b)/3 (u.f) 1 (eq. 14).  The forcing is a polynomial of second degree in c_i, so its
// moments are f (modes 1-3), tr Sigma (4), Sxx - Syy (5), Sxx + Syy - 2 Szz (6), the
// off-diagonal elements (7-9) and zero for the others.  noise (or null): numbers added to the
// modes k >= 4 of n* (lb_noise_modes).  emit(q, n*_q) takes the results.
template <typename Emit>
__device__ __forceinline__ void mrt_collide(const double *n, double rho, double ux, double uy, double uz, double fx,
                                            double fy, double fz, const Rep &R, const double *noise, Emit emit)
{
    const double gs = R.gamma_s, gb = R.gamma_b, gg = R.gamma_ghost;
    const double uu = ux * ux + uy * uy + uz * uz, uf = ux * fx + uy * fy + uz * fz;
    // Sigma (symmetric)
    const double as = 0.5 * (1.0 + gs), ab = (1.0 + gb) / 3.0;
    const double sxx = as * (2.0 * ux * fx - 2.0 / 3.0 * uf) + ab * uf;
    const double syy = as * (2.0 * uy * fy - 2.0 / 3.0 * uf) + ab * uf;
    const double szz = as * (2.0 * uz * fz - 2.0 / 3.0 * uf) + ab * uf;
    const double sxy = as * (ux * fy + uy * fx), sxz = as * (ux * fz + uz * fx), syz = as * (uy * fz + uz * fy);
    const double mf[10] = {0.0, fx, fy, fz, sxx + syy + szz, sxx - syy, sxx + syy - 2.0 * szz, sxy, sxz, syz};
    // n_eq = rho w (ev +- od), and the pairs' sums and differences of n - n_eq
    const double ev0 = 1.0 - 1.5 * uu;
    auto equilibrium = [&](int q, double &ev, double &od) {
        const double cu = kCx[q] * ux + kCy[q] * uy + kCz[q] * uz;
        ev = ev0 + 4.5 * cu * cu;
        od = 3.0 * cu;
    };
    double dn[19];
    dn[0] = n[0] - rho * lb_w(0) * ev0;
#pragma unroll
    for (int p = 1; p < 10; ++p) {
        const int q = 2 * p - 1;
        double ev, od;
        equilibrium(q, ev, od);
        const double rw = rho * lb_w(q), da = n[q] - rw * (ev + od), db = n[q + 1] - rw * (ev - od);
        dn[q] = da + db;
        dn[q + 1] = da - db;
    }
    double ms[19];
#pragma unroll
    for (int k = 0; k < 19; ++k) {
        double m = 0.0;
        bool first = true;
        if (!mrt_odd(k)) {
            m = kMrt.e[k][0] * dn[0];
            first = kMrt.e[k][0] == 0.0;
        }
#pragma unroll
        for (int p = 1; p < 10; ++p) {
            const double e = kMrt.e[k][2 * p - 1], v = dn[mrt_odd(k) ? 2 * p : 2 * p - 1];
            if (e == 0.0) continue;
            m = first ? e * v : m + e * v;
            first = false;
        }
        const double g = k <= 3 ? 1.0 : (k == 4 ? gb : (k <= 9 ? gs : gg));
        if (k > 0 && k < 10) m = g * m + mf[k];
        else if (k > 0) m *= g;
        ms[k] = m * kMrt.binv[k];
        if (noise && k >= 4) ms[k] += noise[k];
    }
    asm volatile("" : "+v"(ux), "+v"(uy), "+v"(uz));   // computed again: 19 values fewer kept
    emit(0, lb_w(0) * (rho * ev0 + mrt_back<0, false>(ms, 0)));
#pragma unroll
    for (int p = 1; p < 10; ++p) {
        const int q = 2 * p - 1;
        double ev, od;
        equilibrium(q, ev, od);
        const double a = rho * ev + mrt_back<0, false>(ms, q), b = rho * od + mrt_back<0, true>(ms, q);
        emit(q, lb_w(q) * (a + b));
        emit(q + 1, lb_w(q) * (a - b));
    }
}

// Mode noise of eq. 13 for site i of replica r: mode k >= 4 receives phi_k r_k, phi_k = sqrt(rho kT
// b_k (1 - gamma_k^2) / c_s^2), carried to the populations as w_q e_k(c_q) a_k, a_k = phi_k r_k /
// b_k.  kT = dt^2 / Omega in LB units; gamma_k of the collision (BGK: 1 - 1/tau for every
// non-conserved mode).  r_k are the normal numbers of purposes 0-3 (mode k takes number k - 4).
__device__ __forceinline__ void lb_noise_modes(const Rep &R, int r, long long i, unsigned long long step, double rho,
                                               double *a)
{
    const double rk = 3.0 * fmax(rho, 0.0) * (R.dt * R.dt / R.omega);
    const bool mrt = R.lb_mode == HSF_LB_MRT;
    const double gbgk = 1.0 - 1.0 / R.tau;
    const double gb = mrt ? R.gamma_b : gbgk, gs = mrt ? R.gamma_s : gbgk, gg = mrt ? R.gamma_ghost : gbgk;
    const double sb = sqrt(rk * (1.0 - gb * gb)), ss = sqrt(rk * (1.0 - gs * gs)), sg = sqrt(rk * (1.0 - gg * gg));
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        double z[4];
        normals4(R.seed, (uint64_t)r, (uint64_t)i, step, (uint64_t)p, z);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 4 + 4 * p + j;
            if (k < 19) a[k] = (k == 4 ? sb : (k <= 9 ? ss : sg)) * (kMrt.rbinv[k] * z[j]);
        }
    }
}

// One LB step, push form: read the 19 pre-collision populations of this site,
// take the moments of eq. 9 (u with the half-force shift), relax towards the
// equilibrium of eq. 11 with rate 1/tau, add the forcing term
//   F_i = (1 - 1/(2 tau)) w_i [3 (c_i - u).f + 9 (c_i.u)(c_i.f)],
// and write each post-collision population to the neighbour it streams to.  NOISE adds
// the mode noise of eq. 13 before streaming.  MODE: HSF_LB_BGK or HSF_LB_MRT when every
// replica uses that collision (each variant needs only its own registers), -1 for a batch
// that mixes them (chosen per replica).
//
// Without noise bound by memory: 152 B (FP32 populations) or 304 B per site and 24 B of force;
// 128^3 FP32 with density and velocity (another 32 B, written by a call's last step only) 86 us,
// 5.0 TB/s, without 75 us.  MRT the same: with all 19 x 19 products written out it took 143
// against BGK's 97 us for four steps of a 64^3 FP64 box and its copies, now 94 against 93.  With
// noise bound by the 16 normal numbers of a site (Philox's integer products, log, sqrt, sincos):
// 64^3 FP64 MRT 34 us against 46 with the full products, 15 square roots and 7
// multiplications per 128-bit product.  Up to 128 registers, four wavefronts per SIMD, where
// the variant has that few.
template <bool NOISE, int MODE, typename pop_t>
__global__ __launch_bounds__(kBlock, NOISE && MODE != HSF_LB_MRT ? 3 : 4) void k_lb(const int *__restrict__ blk_rep, const int *__restrict__ blk_first,
                                               const Rep *__restrict__ rep, const pop_t *__restrict__ nsrc,
                                               pop_t *__restrict__ ndst, const double *__restrict__ f,
                                               double *__restrict__ rho_out, double *__restrict__ u_out,
                                               unsigned long long step, int *__restrict__ bad)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    int x, y, z;
    site_xyz(R, i, x, y, z);
    const long long base = 19LL * R.site_off, vo = 3LL * R.site_off;
    double n[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) n[q] = pop_load(nsrc, base + q * V + i, q);
    double fx = 0.0, fy = 0.0, fz = 0.0;
    if (f) {
        fx = f[vo + i];
        fy = f[vo + V + i];
        fz = f[vo + 2 * V + i];
    }
    double rho = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        rho += n[q];
        jx += kCx[q] * n[q];
        jy += kCy[q] * n[q];
        jz += kCz[q] * n[q];
    }
    const double ux = (jx + 0.5 * fx) / rho, uy = (jy + 0.5 * fy) / rho, uz = (jz + 0.5 * fz) / rho;
    // a non-finite population or force shows in the moments; the host rolls the step back
    if (bad && !(isfinite(rho) && isfinite(ux) && isfinite(uy) && isfinite(uz))) bad[0] = 1;
    double am[19];
    if (NOISE) lb_noise_modes(R, sr.r, i, step, rho, am);
    auto emit = [&](int q, double v) {
        const int xd = wrap1(x + kCx[q], R.Lx), yd = wrap1(y + kCy[q], R.Ly), zd = wrap1(z + kCz[q], R.Lz);
        pop_store(ndst, base + q * V + sidx(R, xd, yd, zd), q, v);
    };
    if (MODE == HSF_LB_MRT || (MODE < 0 && R.lb_mode == HSF_LB_MRT)) {
        mrt_collide(n, rho, ux, uy, uz, fx, fy, fz, R, NOISE ? am : nullptr, emit);
    } else {
        const double om = 1.0 / R.tau, fp = 1.0 - 0.5 / R.tau;
        const double uu = ux * ux + uy * uy + uz * uz;
        const double uf = ux * fx + uy * fy + uz * fz;
        double even = 0.0, odd = 0.0;   // the noise of a pair of opposite velocities
#pragma unroll
        for (int q = 0; q < 19; ++q) {
            const double cu = kCx[q] * ux + kCy[q] * uy + kCz[q] * uz;
            const double cf = kCx[q] * fx + kCy[q] * fy + kCz[q] * fz;
            const double wq = lb_w(q);
            const double neq = rho * wq * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
            const double F = fp * wq * (3.0 * (cf - uf) + 9.0 * cu * cf);
            double v = n[q] - om * (n[q] - neq) + F;
            if (NOISE) {
                const bool lower = q > 0 && q % 2 == 0;   // the second of a pair
                if (!lower) even = mrt_back<4, false>(am, q);
                if (!lower && q > 0) odd = mrt_back<4, true>(am, q);
                v += wq * (q == 0 ? even : (lower ? even - odd : even + odd));
            }
            emit(q, v);   // stored at once: fewer live registers
        }
    }
    if (!rho_out) return;   // a later step of the call writes them
    rho_out[R.site_off + i] = rho;
    u_out[vo + i] = ux;
    u_out[vo + V + i] = uy;
    u_out[vo + 2 * V + i] = uz;
}

// Conservative convection-diffusion update.  Face between r and r + e_a:
//   J = dt * (-(phi_r + phi_e)/2 (mu_e - mu_r))
//     + [(phi_r + phi_e)/2 - ((phi u_a)_e - (phi u_a)_r)/2] (u_a,r + u_a,e)/2
// phi_new(r) = phi(r) - sum_a (J(r + e_a/2) - J(r - e_a/2)).
// NOISE adds the composition noise of eq. 5 as a random flux on every bond, drawn
// beforehand by k_cd_noise into jn.
// Columns as in k_mu: z neighbours are the lane's other planes, x neighbours come from the
// adjacent lanes, the rows y +- 1 are loaded (23 loads per site for 3 species, against 44 with
// one site per lane, which took 74 us at 128^3 for 201 MB; now 46 us, 4.4 TB/s).  4 x 256 x 256 in
// calls as above: 61, 25 and 12.5 us.
template <bool NOISE, int NSP, int P, bool SHORT>
__global__ __launch_bounds__(kBlock) void k_cd(const int *__restrict__ blk_rep, const int *__restrict__ blk_first,
                                               const Rep *__restrict__ rep, const double *__restrict__ phi,
                                               const double *__restrict__ mu, const double *__restrict__ u,
                                               double *__restrict__ phi_out, const double *__restrict__ jn,
                                               double diff_scale, int *__restrict__ bad)
{
    typedef Sites<double, P> row_t;
    constexpr int CZ = kCdZ;
    Col<P, CZ, SHORT> t;
    if (!t.init(blk_rep, blk_first, rep)) return;
    const Rep &R = rep[t.r];
    const long long fo = off_field(R, NSP), vo = 3LL * R.site_off;
    const double dt = R.dt * diff_scale;   // diffusive flux over dt (or dt/2 in the CN step)
    // the velocity at the core planes' sites and their neighbours along each axis (l, c, h),
    // shared by the species
    row_t ul[3][CZ], uc[3][CZ], uh[3][CZ];
    if (u) {
        const double *ux = u + vo, *uy = ux + t.V, *uz = uy + t.V;
        row_t zz[CZ + 2];
#pragma unroll
        for (int q = 0; q < CZ + 2; ++q) zz[q] = t.load(uz, t.z(q) + t.row);
#pragma unroll
        for (int j = 0; j < CZ; ++j) {
            const long long zq = t.z(j + 1);
            uc[0][j] = t.load(ux, zq + t.row);
            ul[1][j] = t.load(uy, zq + t.dn);
            uc[1][j] = t.load(uy, zq + t.row);
            uh[1][j] = t.load(uy, zq + t.up);
            ul[2][j] = zz[j];
            uc[2][j] = zz[j + 1];
            uh[2][j] = zz[j + 2];
        }
#pragma unroll
        for (int j = 0; j < CZ; ++j) x_pair<P>(uc[0][j], ul[0][j], uh[0][j]);
    }
#pragma unroll 1
    for (int I = 0; I < NSP; ++I) {
        const double *f = phi + fo + (long long)I * t.V, *g = mu + fo + (long long)I * t.V;
        row_t pz[CZ + 2], mz[CZ + 2];
#pragma unroll
        for (int q = 0; q < CZ + 2; ++q) {
            const long long zq = t.z(q) + t.row;
            pz[q] = t.load(f, zq);
            mz[q] = t.load(g, zq);
        }
        row_t pl[CZ], ph[CZ], ml[CZ], mh[CZ];   // y neighbours
#pragma unroll
        for (int j = 0; j < CZ; ++j) {
            const long long zq = t.z(j + 1);
            pl[j] = t.load(f, zq + t.dn);
            ph[j] = t.load(f, zq + t.up);
            ml[j] = t.load(g, zq + t.dn);
            mh[j] = t.load(g, zq + t.up);
        }
        const double *jI = NOISE ? jn + 3 * fo + 3 * (long long)I * t.V : nullptr;
#pragma unroll
        for (int j = 0; j < CZ; ++j) {
            row_t xl, xh, yl, yh;   // x neighbours of phi and mu
            x_pair<P>(pz[j + 1], xl, xh);
            x_pair<P>(mz[j + 1], yl, yh);
            row_t nl[3], nh[3];     // noise fluxes of the lower and upper faces
            if (NOISE) {
                const long long zq = t.z(j + 1);
                row_t dummy;
                nh[0] = t.load(jI, zq + t.row);
                x_pair<P>(nh[0], nl[0], dummy);
                nh[1] = t.load(jI, t.V + zq + t.row);
                nl[1] = t.load(jI, t.V + zq + t.dn);
                nh[2] = t.load(jI, 2 * t.V + zq + t.row);
                nl[2] = t.load(jI, 2 * t.V + t.z(j) + t.row);
            }
            row_t out;
#pragma unroll
            for (int e = 0; e < P; ++e) {
                const double pr = pz[j + 1].s[e], mr = mz[j + 1].s[e];
                const double pn_l[3] = {xl.s[e], pl[j].s[e], pz[j].s[e]}, pn_h[3] = {xh.s[e], ph[j].s[e], pz[j + 2].s[e]};
                const double mn_l[3] = {yl.s[e], ml[j].s[e], mz[j].s[e]}, mn_h[3] = {yh.s[e], mh[j].s[e], mz[j + 2].s[e]};
                double div = 0.0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    // face between lo and r, then between r and hi
                    const double lo = pn_l[a], hi = pn_h[a];
                    double jl = dt * (-0.5 * (lo + pr) * (mr - mn_l[a]));
                    double jh = dt * (-0.5 * (pr + hi) * (mn_h[a] - mr));
                    if (u) {
                        const double vl = ul[a][j].s[e], vc = uc[a][j].s[e], vh = uh[a][j].s[e];
                        jl += (0.5 * (lo + pr) - 0.5 * (pr * vc - lo * vl)) * (0.5 * (vl + vc));
                        jh += (0.5 * (pr + hi) - 0.5 * (hi * vh - pr * vc)) * (0.5 * (vc + vh));
                    }
                    if (NOISE) {
                        jl += nl[a].s[e];
                        jh += nh[a].s[e];
                    }
                    div += jh - jl;
                }
                out.s[e] = pr - div;
            }
            if (t.core && j < t.nz) {
#pragma unroll
                for (int e = 0; e < P; ++e)
                    if (bad && !isfinite(out.s[e])) bad[0] = 1;
                t.store(phi_out, fo + (long long)I * t.V + (long long)(t.z0 + j) * t.plane + t.row, out);
            }
        }
    }
}

// Composition noise of eq. 5 as random bond fluxes: the bond between site s and
// s + e_a of species I carries jn = sqrt(2 dt max(phi_bond, 0) / Omega) g with
// phi_bond = (phi_I(s) + phi_I(s + e_a)) / 2 and g number a of the normal numbers of
// (site s, purpose 4 + I).  Its divergence conserves each species exactly and has the
// covariance (2 dt / Omega)(-div phi grad) of eq. 5 over a step.
// Layout of jn: per replica [species][3][V] at 3 nsp site_off.
__global__ __launch_bounds__(kBlock) void k_cd_noise(const int *__restrict__ blk_rep,
                                                     const int *__restrict__ blk_first,
                                                     const Rep *__restrict__ rep, Chain ch,
                                                     const double *__restrict__ phi, double *__restrict__ jn,
                                                     unsigned long long step)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
    int x, y, z;
    site_xyz(R, i, x, y, z);
    const long long fo = off_field(R, ch.nsp);
    const long long up[3] = {sidx(R, wrap1(x + 1, R.Lx), y, z), sidx(R, x, wrap1(y + 1, R.Ly), z),
                             sidx(R, x, y, wrap1(z + 1, R.Lz))};
    for (int I = 0; I < ch.nsp; ++I) {
        const double *p = phi + fo + I * V;
        double g[4];
        normals4(R.seed, (uint64_t)sr.r, (uint64_t)i, step, (uint64_t)(4 + I), g);
        const double pr = p[i];
#pragma unroll
        for (int a = 0; a < 3; ++a)
            jn[3 * fo + (3 * I + a) * V + i] = sqrt(2.0 * R.dt * fmax(0.5 * (pr + p[up[a]]), 0.0) / R.omega) * g[a];
    }
}

// Fluid at rest with density 1: n_i = w_i.
template <typename pop_t>
__global__ __launch_bounds__(kBlock) void k_lb_rest(const int *__restrict__ blk_rep,
                                                    const int *__restrict__ blk_first, const Rep *__restrict__ rep,
                                                    pop_t *__restrict__ n)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
#pragma unroll
    for (int q = 0; q < 19; ++q) pop_store(n, 19LL * R.site_off + q * V + i, q, lb_w(q));
}

// FP64 populations to the FP32 deviation storage (to_f32) or back.
__global__ __launch_bounds__(kBlock) void k_lb_convert(const int *__restrict__ blk_rep,
                                                       const int *__restrict__ blk_first,
                                                       const Rep *__restrict__ rep, int to_f32,
                                                       const void *__restrict__ src, void *__restrict__ dst)
{
    const SiteRef sr = site_ref(blk_rep, blk_first);
    const Rep &R = rep[sr.r];
    const long long V = R.V, i = sr.i;
    if (i >= V) return;
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const long long k = 19LL * R.site_off + q * V + i;
        if (to_f32) pop_store((float *)dst, k, q, ((const double *)src)[k]);
        else ((double *)dst)[k] = pop_load((const float *)src, k, q);
    }
}

void launch_mu(hipStream_t s, const Plan &p, int P, const Rep *rep, Chain ch, const double *phi, const double *w,
               double *mu)
{
    auto kern = P == 2   ? (ch.nsp == 3 ? k_mu<3, 2, false> : k_mu<2, 2, false>)
                : P == 1 ? (ch.nsp == 3 ? k_mu<3, 1, false> : k_mu<2, 1, false>)
                         : (ch.nsp == 3 ? k_mu<3, 1, true> : k_mu<2, 1, true>);
    hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, phi, w, mu);
}

void launch_force(hipStream_t s, const Plan &p, const Rep *rep, Chain ch, const double *phi, const double *mu,
                  double *f)
{
    hipLaunchKernelGGL(k_force, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, ch, phi, mu, f);
}

template <typename pop_t>
static void launch_lb_t(hipStream_t s, const Plan &p, const Rep *rep, const pop_t *nsrc, pop_t *ndst,
                        const double *f, double *rho, double *u, bool noise, unsigned long long step, int lb_mode,
                        hipEvent_t e0, hipEvent_t e1, int *bad)
{
    auto pick = [&](auto bgk, auto mrt, auto mixed) { return lb_mode == HSF_LB_BGK ? bgk : lb_mode == HSF_LB_MRT ? mrt : mixed; };
    auto kern = noise ? pick(k_lb<true, HSF_LB_BGK, pop_t>, k_lb<true, HSF_LB_MRT, pop_t>, k_lb<true, -1, pop_t>)
                      : pick(k_lb<false, HSF_LB_BGK, pop_t>, k_lb<false, HSF_LB_MRT, pop_t>, k_lb<false, -1, pop_t>);
    if (e0)
        hipExtLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, e0, e1, 0, p.blk_rep, p.blk_first, rep,
                              nsrc, ndst, f, rho, u, step, bad);
    else
        hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, nsrc, ndst, f,
                           rho, u, step, bad);
}

void launch_lb(hipStream_t s, const Plan &p, const Rep *rep, const void *nsrc, void *ndst, bool f32, const double *f,
               double *rho, double *u, bool noise, unsigned long long step, int lb_mode, hipEvent_t e0,
               hipEvent_t e1, int *bad)
{
    if (f32)
        launch_lb_t<float>(s, p, rep, (const float *)nsrc, (float *)ndst, f, rho, u, noise, step, lb_mode, e0, e1,
                           bad);
    else
        launch_lb_t<double>(s, p, rep, (const double *)nsrc, (double *)ndst, f, rho, u, noise, step, lb_mode, e0,
                            e1, bad);
}

void launch_lb_convert(hipStream_t s, const Plan &p, const Rep *rep, bool to_f32, const void *src, void *dst)
{
    hipLaunchKernelGGL(k_lb_convert, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep,
                       to_f32 ? 1 : 0, src, dst);
}

void launch_cd(hipStream_t s, const Plan &p, int P, const Plan &ps, const Rep *rep, Chain ch, const double *phi,
               const double *mu, const double *u, double *phi_out, double *noise_flux, unsigned long long step,
               hipEvent_t e0, hipEvent_t e1, double diff_scale, int *bad)
{
    // with noise the events bracket both kernels: e0 at the start of the flux draw
    if (noise_flux) {
        if (e0)
            hipExtLaunchKernelGGL(k_cd_noise, dim3(ps.nblocks), dim3(kBlock), 0, s, e0, nullptr, 0, ps.blk_rep,
                                  ps.blk_first, rep, ch, phi, noise_flux, step);
        else
            hipLaunchKernelGGL(k_cd_noise, dim3(ps.nblocks), dim3(kBlock), 0, s, ps.blk_rep, ps.blk_first, rep, ch,
                               phi, noise_flux, step);
        e0 = nullptr;
    }
    auto pick = [&](auto noise) {
        constexpr bool N = noise();
        return P == 2   ? (ch.nsp == 3 ? k_cd<N, 3, 2, false> : k_cd<N, 2, 2, false>)
               : P == 1 ? (ch.nsp == 3 ? k_cd<N, 3, 1, false> : k_cd<N, 2, 1, false>)
                        : (ch.nsp == 3 ? k_cd<N, 3, 1, true> : k_cd<N, 2, 1, true>);
    };
    auto kern = noise_flux ? pick(std::true_type()) : pick(std::false_type());
    if (e0 || e1)
        hipExtLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, e0, e1, 0, p.blk_rep, p.blk_first, rep, phi,
                              mu, u, phi_out, noise_flux, diff_scale, bad);
    else
        hipLaunchKernelGGL(kern, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep, phi, mu, u,
                           phi_out, noise_flux, diff_scale, bad);
}

void launch_lb_rest(hipStream_t s, const Plan &p, const Rep *rep, void *n, bool f32)
{
    if (f32)
        hipLaunchKernelGGL(k_lb_rest<float>, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep,
                           (float *)n);
    else
        hipLaunchKernelGGL(k_lb_rest<double>, dim3(p.nblocks), dim3(kBlock), 0, s, p.blk_rep, p.blk_first, rep,
                           (double *)n);
}

}  // namespace hsf
