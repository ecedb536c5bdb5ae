// prop_rows.hip -- paired propagator sweeps of K contour steps per launch (eq. 16-17).
//
// What bounds the one-step kernels is not arithmetic: a launch moves every propagator,
// field factor and density term once per contour step and is short enough for launch
// and memory latency to matter.  Here a workgroup keeps a CY x CZ bundle of whole x rows
// (with a halo of K rows per side) in registers for K steps, so a step's input and field
// factor are read once per K steps.  One wavefront owns one y row: its 64 lanes are P
// consecutive x sites each and its registers the row's CZ + 2K planes in z.  Neighbours in
// z are the lane's own registers, neighbours in x come from the adjacent lanes (wavefront
// rotations) and neighbours in y from the adjacent wavefronts through LDS (each row is
// written once and read twice per step, 64 lanes consecutive: no bank conflicts).  Boxes
// of exactly 64 P sites in x need no x halo, the rotation closes the periodic row; other
// boxes are cut into row pieces of at most 64 - 2K sites with K halo sites per side.
// Halo rows are recomputed by the neighbouring workgroups.
//
// Every stored value is the same expression of the same operands, in the same order, as
// in the one-step kernels, so the densities are bit for bit those of the one-step
// sequence (up to the order of Q's sum over workgroups).
//
// Measured against the one-step paired kernels (hsf_evaluate calls with device buffers, the best
// tiling of each kind): FP32 64^3 pair 116 against 179 us (4 launches of 16.2 us for 16 of 8.0 us), 96^3
// 203 / 228, 128^3 221 / 308 (6 of 22.4 for 12 of 18.4), 192^3 1040 / 1300, 12 solutions of
// 32^3 to 64^3 205 / 271; FP64 64^3 pair 160 / 231, 128^3 419 / 506 (6 of 48.0 for 12 of 31.5).
// At 128^3 a launch of the 128x8x4 K = 2 bundle moves 94 MB by the counters (20.3 us inside an
// inversion, 4.6 TB/s) with the vector units issuing 37 % of the time: it is bound by the latency
// of its phases (load, step, step, store) and by bytes, about equally.
#include <hip/hip_ext.h>

#include "device_common.h"
#include "prop_rows.h"

namespace hsf {

// Global memory through buffer descriptors: a uniform base and byte offset (scalar
// registers) plus the lane's own offset, so a row costs one instruction and no address
// arithmetic, and a lane whose offset lies past the end (kOutside) reads zero and stores
// nothing, so rows need no branches for the lanes outside a piece.  Arrays reached this way
// are smaller than 2^31 bytes.
constexpr unsigned kOutside = 0x80000000u;
typedef __amdgpu_buffer_rsrc_t buf_t;

__device__ __forceinline__ buf_t make_buf(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x20000);
}

template <typename T>
__device__ __forceinline__ T buf_load(buf_t b, unsigned lane_off, int off)
{
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, lane_off, off, 0));
    else if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, lane_off, off, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(b, lane_off, off, 0));
}
template <typename T>
__device__ __forceinline__ void buf_store(buf_t b, unsigned lane_off, int off, const T &v)
{
    if constexpr (sizeof(T) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, lane_off, off, 0);
    else if constexpr (sizeof(T) == 8) {
        typedef unsigned v2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2, v), b, lane_off, off, 0);
    } else {
        typedef unsigned v4 __attribute__((ext_vector_type(4)));
        // The data registers of a store wider than 64 bits must not be written by the next
        // vector instructions.  The compiler keeps that distance except for stores with a
        // scalar offset register, which this chip does not excuse (8 lanes of a row came out
        // with the overwritten values now and then), so the offset goes through the lane's.
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4, v), b, lane_off + (unsigned)off, 0, 0);
    }
}

// The tile of a workgroup and the wavefront's part of it.  All but the lane offsets is
// uniform; zo[q] is the byte offset of region plane q at the wavefront's row.
template <typename real, int P, int K, int CY, int CZ>
struct RowsTile {
    static constexpr int NY = CY + 2 * K, NZ = CZ + 2 * K;
    int r, pb, V, bytes;         // replica, plan block, sites and bytes of one propagator
    int w, lane;                 // wavefront (= region row), lane
    int nzc;                     // core planes of this row inside the box (0: no core row)
    int zo[NZ];
    unsigned xl, xc;             // the lane's byte offset for loads, and as a core site (else kOutside)
    real c0, c1, c2, c3, csum;
};

template <typename real>
__device__ __forceinline__ real scale_of(const RepState *st, int r, int s)
{
    return (real)ldexp(1.0, -st[r].scale_e[s - 1]);
}

__device__ __forceinline__ int species_of(unsigned long long types, int s) { return (int)((types >> (s - 1)) & 1ull); }

// Level k of a sweep (k = 1 .. K): the stencil of v on the region shrunk by k rows per
// side, then the step's product; core sites are stored.  Recursive in k so that every
// register index is a constant.
template <typename real, int P, int K, int CY, int CZ, bool FWD, int k>
__device__ __forceinline__ void rows_level(const RowsTile<real, P, K, CY, CZ> &t, const RowsHalf &h,
                                           unsigned long long types, int N, const RepState *__restrict__ st,
                                           const real *__restrict__ E, real *G, Sites<real, P> (&v)[CZ + 2 * K],
                                           Sites<real, P> (&ev)[CZ + 2 * K - 2], double (&gsum)[K + 1], int sums,
                                           Sites<real, P> *lds)
{
    typedef Sites<real, P> row_t;
    constexpr int NY = CY + 2 * K, NZ = CZ + 2 * K;
    if constexpr (k <= K) {
        if (k > h.n) return;
        const int s = FWD ? h.first + k - 1 : h.first - k + 1;
        const int w = t.w;
        const bool work = w >= k && w < NY - k;   // the wavefront computes at this level
        const buf_t slot = make_buf(G + (long long)(s - 1) * t.V, t.bytes);
        // loads of this level: the field factors when the species changed ...
        const int ts = species_of(types, s);
        if (k > 1 && work && ts != species_of(types, FWD ? s - 1 : s + 1)) {
            const buf_t e = make_buf(E + (long long)ts * t.V, t.bytes);
#pragma unroll
            for (int q = k; q < NZ - k; ++q) ev[q - 1] = buf_load<row_t>(e, t.xl, t.zo[q]);
        }
        // ... and what multiplies the stored value: at a bead's second visit what the first
        // one left in its slot (csum for bead N, which has no stencil), else 1
        row_t sl[CZ];
        const real one = h.late ? t.csum : (real)1;
#pragma unroll
        for (int j = 0; j < CZ; ++j)
#pragma unroll
            for (int u = 0; u < P; ++u) sl[j].s[u] = one;
        if (h.late && t.nzc && (!FWD || s < N)) {
#pragma unroll
            for (int j = 0; j < CZ; ++j) sl[j] = buf_load<row_t>(slot, t.xc, t.zo[K + j]);
        }
        const real sc = scale_of<real>(st, t.r, s);
        // publish the rows of level k - 1
        if (k > 1) __syncthreads();   // the reads of the level before are done
        if (w >= k - 1 && w <= NY - k) {
            row_t *mine = lds + (w * NZ) * 64 + t.lane;
#pragma unroll
            for (int q = k - 1; q <= NZ - k; ++q) mine[q * 64] = v[q];
        }
        __syncthreads();
        if (work) {
            const row_t *ym = lds + ((w - 1) * NZ) * 64 + t.lane, *yp = lds + ((w + 1) * NZ) * 64 + t.lane;
            row_t a0[3], a1[3], a2[3];
#pragma unroll
            for (int q = k - 1; q <= NZ - k; ++q) {
                // in-plane class sums of plane q: centre, 4 edge-sharing, 4 corner neighbours
                const row_t c = v[q], m = ym[q * 64], p = yp[q * 64];
                const row_t ec = x_sums(c), em = x_sums(m), ep = x_sums(p);
                const int i = q % 3;
#pragma unroll
                for (int u = 0; u < P; ++u) {
                    a0[i].s[u] = c.s[u];
                    a1[i].s[u] = ec.s[u] + (m.s[u] + p.s[u]);
                    a2[i].s[u] = em.s[u] + ep.s[u];
                }
                if (q < k + 1) continue;
                const int o = q - 1;   // output plane
                const int il = (o - 1) % 3, ic = o % 3, ih = (o + 1) % 3;
                row_t S, g;
#pragma unroll
                for (int u = 0; u < P; ++u) {
                    S.s[u] = t.c0 * a0[ic].s[u] + t.c1 * (a1[ic].s[u] + (a0[il].s[u] + a0[ih].s[u])) +
                             t.c2 * (a2[ic].s[u] + (a1[il].s[u] + a1[ih].s[u])) + t.c3 * (a2[il].s[u] + a2[ih].s[u]);
                    g.s[u] = ev[o - 1].s[u] * S.s[u] * sc;
                }
                v[o] = g;
                if (o >= K && o < K + CZ) {
                    const int j = o - K;
                    row_t val;
#pragma unroll
                    for (int u = 0; u < P; ++u) val.s[u] = FWD ? g.s[u] * sl[j].s[u] : sl[j].s[u] * S.s[u];
                    buf_store(slot, j < t.nzc ? t.xc : kOutside, t.zo[o], val);
                }
            }
        }
        if (FWD && (sums || s == N) && t.nzc) {   // core sum of the stored G_s
#pragma unroll
            for (int j = 0; j < CZ; ++j)
#pragma unroll
                for (int u = 0; u < P; ++u)
                    if (j < t.nzc && t.xc != kOutside) gsum[k] += (double)v[K + j].s[u];
        }
        rows_level<real, P, K, CY, CZ, FWD, k + 1>(t, h, types, N, st, E, G, v, ev, gsum, sums, lds);
    }
}

template <typename real, int P, int K, int CY, int CZ, bool FWD>
__device__ __forceinline__ void rows_half(const RowsTile<real, P, K, CY, CZ> &t, const Rep &R, const RowsHalf &h,
                                          unsigned long long types, int N, const RepState *__restrict__ st,
                                          PropBufs<real> b, const real *__restrict__ in, real *__restrict__ out,
                                          double *__restrict__ partG, int nblocks, int sums, int act,
                                          Sites<real, P> *lds)
{
    typedef Sites<real, P> row_t;
    constexpr int NY = CY + 2 * K, NZ = CZ + 2 * K;
    real *G = b.G + (long long)N * R.site_off;
    const real *E = b.E + off_poly(R);
    const int w = t.w, s1 = h.first;   // bead of the first level
    row_t v[NZ];                       // the propagator on the lane's column
    row_t ev[NZ - 2];                  // field factors of planes 1 .. NZ - 2
    double gsum[K + 1], esum[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k <= K; ++k) gsum[k] = 0.0;
    // the launch's first loads: the propagator on the whole region, the field factors of
    // the first level on the rows that compute it
    const int sb = FWD ? 1 : N;   // the bead the sweep starts from
    const real *src = h.start ? E + (long long)species_of(types, sb) * t.V
                              : (FWD && !h.from_pp ? G + (long long)(s1 - 2) * t.V : in + R.site_off);
    const buf_t vb = make_buf(src, t.bytes);
#pragma unroll
    for (int q = 0; q < NZ; ++q) v[q] = buf_load<row_t>(vb, t.xl, t.zo[q]);
    if (h.n > 0 && w >= 1 && w < NY - 1) {
        const buf_t e = make_buf(E + (long long)species_of(types, s1) * t.V, t.bytes);
#pragma unroll
        for (int q = 1; q < NZ - 1; ++q) ev[q - 1] = buf_load<row_t>(e, t.xl, t.zo[q]);
    }
    if (!act) return;   // uniform for the block
    if (h.start) {
        // G_1 = E csum sc_1, G+_N = E csum sc_N (sigma of the constant 1 is csum)
        const real sc = scale_of<real>(st, t.r, sb);
#pragma unroll
        for (int q = 0; q < NZ; ++q)
#pragma unroll
            for (int u = 0; u < P; ++u) v[q].s[u] = v[q].s[u] * t.csum * sc;
        const buf_t slot = make_buf(G + (long long)(sb - 1) * t.V, t.bytes);
        if (FWD) {
#pragma unroll
            for (int j = 0; j < CZ; ++j) buf_store(slot, j < t.nzc ? t.xc : kOutside, t.zo[K + j], v[K + j]);
            if (sums) {
                const buf_t ea = make_buf(E, t.bytes), eb = make_buf(E + t.V, t.bytes);
#pragma unroll
                for (int j = 0; j < CZ; ++j) {
                    if (j >= t.nzc || t.xc == kOutside) continue;
                    const row_t x = buf_load<row_t>(ea, t.xc, t.zo[K + j]), y = buf_load<row_t>(eb, t.xc, t.zo[K + j]);
#pragma unroll
                    for (int u = 0; u < P; ++u) {
                        gsum[0] += (double)v[K + j].s[u];
                        esum[0] += (double)x.s[u];
                        esum[1] += (double)y.s[u];
                    }
                }
            }
        } else if (h.late) {   // bead N's term, when the forward sweep has passed it already
#pragma unroll
            for (int j = 0; j < CZ; ++j) {
                const unsigned xc = j < t.nzc ? t.xc : kOutside;
                row_t gs = buf_load<row_t>(slot, xc, t.zo[K + j]);
#pragma unroll
                for (int u = 0; u < P; ++u) gs.s[u] = gs.s[u] * t.csum;
                buf_store(slot, xc, t.zo[K + j], gs);
            }
        }
    }
    rows_level<real, P, K, CY, CZ, FWD, 1>(t, h, types, N, st, E, G, v, ev, gsum, sums, lds);
    if (h.out && t.nzc) {   // the last propagator for the next launch
        const buf_t ob = make_buf(out + R.site_off, t.bytes);
#pragma unroll
        for (int j = 0; j < CZ; ++j) buf_store(ob, j < t.nzc ? t.xc : kOutside, t.zo[K + j], v[K + j]);
    }
    if (!FWD) return;
    // partial sums of the stored G_s over the core: every step with `sums` (the FP32
    // scales), bead N's always (Q); with `sums` also those of E_A and E_B
    const int s_last = s1 + h.n - 1;
    if (!sums && s_last != N) return;
    __shared__ double ws[NY][K + 3];
#pragma unroll
    for (int k = 0; k <= K; ++k) {
        const double x = wave_sum(gsum[k]);
        if (t.lane == 0) ws[w][k] = x;
    }
    if (sums && h.start) {
        const double x = wave_sum(esum[0]), y = wave_sum(esum[1]);
        if (t.lane == 0) {
            ws[w][K + 1] = x;
            ws[w][K + 2] = y;
        }
    }
    __syncthreads();
    const int k = (int)threadIdx.x;
    if (k > K + 2) return;
    const bool level = k <= K;
    const int s = level ? s1 + k - 1 : 0;                     // bead of the sum (k = 0: G_1)
    const int row = level ? s - 1 : N + (k - K - 1);          // row of partG
    const bool want = level ? ((k == 0 ? h.start && sums : k <= h.n) && (sums || s == N)) : (sums && h.start);
    if (!want) return;
    double x = 0.0;
#pragma unroll
    for (int q = K; q < K + CY; ++q) x += ws[q][k];
    partG[(long long)row * nblocks + t.pb] = x;
}

// One launch: the first info.nf workgroups take the forward half, the rest the backward
// half, each over every tile of the plan.
template <typename real, int P, int K, int CY, int CZ, bool ARGS>
__global__ __launch_bounds__((CY + 2 * K) * 64) __attribute__((amdgpu_waves_per_eu(rows_waves(sizeof(real), P, K, CZ)))) void k_rows(RowsInfo info, const int *__restrict__ blk_rep,
                                                            const int *__restrict__ blk_first,
                                                            const Rep *__restrict__ rep,
                                                            const RepState *__restrict__ st, PropBufs<real> b,
                                                            const real *__restrict__ fin, real *__restrict__ fout,
                                                            const real *__restrict__ gin, real *__restrict__ gout,
                                                            double *__restrict__ partG, int nblocks, int sums,
                                                            ArgReps ar)
{
    constexpr int NY = CY + 2 * K, NZ = CZ + 2 * K;
    __shared__ Sites<real, P> lds[NY * NZ * 64];
    const int pb0 = plan_block();
    const bool fwd = pb0 < info.nf;
    RowsTile<real, P, K, CY, CZ> t;
    Rep R;
    t.pb = fwd ? pb0 : pb0 - info.nf;
    int act, lb;
    if (ARGS) {
        int r = 0;
#pragma unroll
        for (int k = 1; k < kArgReps; ++k)
            if (k < ar.n && t.pb >= ar.blk_first[k]) r = k;
        t.r = r;
        R = r == 0 ? ar.rep[0] : (r == 1 ? ar.rep[1] : (r == 2 ? ar.rep[2] : ar.rep[3]));
        lb = t.pb - ar.blk_first[r];
        act = st[r].active | (ar.n == 1);
    } else {
        t.r = blk_rep[t.pb];
        R = rep[t.r];
        lb = t.pb - blk_first[t.r];
        act = st[t.r].active;
        if (!act) return;
    }
    const RowsCut cut = rows_cut(R.Lx, P, K);
    const int nty = (R.Ly + CY - 1) / CY;
    t.w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    t.lane = (int)threadIdx.x & 63;
    const int x0 = (lb % cut.ntx) * cut.width;
    lb /= cut.ntx;
    const int y0 = (lb % nty) * CY, z0 = (lb / nty) * CZ;
    t.V = (int)R.V;
    t.bytes = t.V * (int)sizeof(real);
    t.nzc = t.w >= K && t.w < K + CY && y0 + t.w - K < R.Ly ? min(CZ, R.Lz - z0) : 0;
    {
        int y = (y0 - K + t.w) % R.Ly, z = (z0 - K) % R.Lz;
        if (y < 0) y += R.Ly;
        if (z < 0) z += R.Lz;
        const int plane = R.Lx * R.Ly;
        int o = z * plane + y * R.Lx;
#pragma unroll
        for (int q = 0; q < NZ; ++q) {
            t.zo[q] = o * (int)sizeof(real);
            o += plane;
            if (++z == R.Lz) {
                z = 0;
                o -= t.V;
            }
        }
    }
    const int xu = x0 - cut.halo + t.lane * P;   // unwrapped
    int x = xu % R.Lx;
    if (x < 0) x += R.Lx;
    // rows of 128 sites are always whole: no lane is masked
    const bool live = P > 1 || t.lane < cut.width + 2 * cut.halo;
    const bool core = P > 1 || (xu >= x0 && xu < x0 + cut.width && xu < R.Lx);
    t.xl = live ? (unsigned)x * (unsigned)sizeof(real) : kOutside;
    t.xc = core ? t.xl : kOutside;
    t.c0 = (real)R.c[0];
    t.c1 = (real)R.c[1];
    t.c2 = (real)R.c[2];
    t.c3 = (real)R.c[3];
    t.csum = (real)R.csum;
    if (fwd)
        rows_half<real, P, K, CY, CZ, true>(t, R, info.f, info.types, info.N, st, b, fin, fout, partG, nblocks, sums,
                                            act, lds);
    else
        rows_half<real, P, K, CY, CZ, false>(t, R, info.g, info.types, info.N, st, b, gin, gout, partG, nblocks, 0,
                                             act, lds);
}

template <typename real, int P, int K, int CY, int CZ>
static void rows_launch(hipStream_t s, const Plan &p, const Rep *rep, RepState *st, const RowsInfo &info, int grid,
                        PropBufs<real> b, const real *fin, real *fout, const real *gin, real *gout, double *partG,
                        int sums, hipEvent_t e0, hipEvent_t e1)
{
    auto kern = p.args.n ? k_rows<real, P, K, CY, CZ, true> : k_rows<real, P, K, CY, CZ, false>;
    const dim3 blk((CY + 2 * K) * 64);
    if (e0)
        hipExtLaunchKernelGGL(kern, dim3(grid), blk, 0, s, e0, e1, 0, info, p.blk_rep, p.blk_first, rep, st, b, fin,
                              fout, gin, gout, partG, p.nblocks, sums, p.args);
    else
        hipLaunchKernelGGL(kern, dim3(grid), blk, 0, s, info, p.blk_rep, p.blk_first, rep, st, b, fin, fout, gin, gout,
                           partG, p.nblocks, sums, p.args);
}

template <typename real>
void launch_rows(const TileCfg &cfg, hipStream_t s, const Plan &p, const Rep *rep, RepState *st, const Chain &ch,
                 const RowsLaunch &l, PropBufs<real> b, const real *fin, real *fout,
                 const real *gin, real *gout, double *partG, int sums, hipEvent_t e0, hipEvent_t e1)
{
    RowsInfo info{};
    info.f = l.f;
    info.g = l.g;
    info.N = ch.N;
    for (int k = 0; k < ch.N; ++k) info.types |= (unsigned long long)(ch.types[k] & 1) << k;
    info.nf = l.has_f ? p.nblocks : 0;
    const int grid = info.nf + (l.has_g ? p.nblocks : 0);
#define HSF_CASE(CX, CY, CZ, K)                                                                              \
    if constexpr (sizeof(real) == 4 || rows_fp64(CX, CY, CZ, K))                                             \
        if (cfg.cx == CX && cfg.cy == CY && cfg.cz == CZ && cfg.k == -K)                                     \
            return rows_launch<real, CX / 64, K, CY, CZ>(s, p, rep, st, info, grid, b, fin, fout, gin, gout, partG, sums, \
                                                     e0, e1);
    HSF_ROWS_CONFIGS(HSF_CASE)
#undef HSF_CASE
}

#define HSF_INST(real)                                                                                        \
    template void launch_rows<real>(const TileCfg &, hipStream_t, const Plan &, const Rep *, RepState *,      \
                                    const Chain &, const RowsLaunch &, PropBufs<real>, const real *,         \
                                    real *, const real *, real *, double *, int, hipEvent_t, hipEvent_t);
HSF_INST(double)
HSF_INST(float)
#undef HSF_INST

}  // namespace hsf
