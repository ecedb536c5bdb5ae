// prop_rows.h -- the row-resident paired sweeps (K contour steps per launch).
#pragma once

#include "prop_block.h"

namespace hsf {

// X(CX, CY, CZ, K): rows of CX = 64 P sites, CY x CZ core rows per workgroup, K steps
// per launch; as a tiling they read {CX, CY, CZ, -K} with K >= 2.
#define HSF_ROWS_CONFIGS(X) \
    X(64, 4, 4, 2)          \
    X(64, 4, 4, 4)          \
    X(64, 8, 4, 2)          \
    X(64, 8, 4, 3)          \
    X(64, 8, 8, 2)          \
    X(64, 8, 8, 3)          \
    X(64, 8, 8, 4)          \
    X(128, 8, 4, 2)         \
    X(128, 8, 8, 3)

inline bool tile_is_rows(const TileCfg &t) { return t.k <= -2; }

// Bundles whose FP64 form fits the registers (about 100 to 165 of them; the others would
// spill) are compiled for both precisions, the others for FP32 only.
constexpr bool rows_fp64(int cx, int cy, int cz, int k)
{
    return cx == 128 ? (k == 2 && cz == 4) : (k == 2 || cz == 4);
}
// Wavefronts per SIMD the registers are limited for (1: no limit).  The 128-site K = 2
// bundle in FP32 fits two workgroups of 12 wavefronts in a CU with at most 80 registers,
// so that one's loads overlap the other's arithmetic: 23.0 against 30.1 us per launch at
// 128^3 with the 93 registers it takes unlimited (one workgroup per CU).
constexpr int rows_waves(size_t rs, int P, int K, int CZ) { return rs == 4 && P == 2 && K == 2 && CZ == 4 ? 6 : 1; }
inline bool rows_fp64(const TileCfg &t) { return rows_fp64(t.cx, t.cy, t.cz, -t.k); }

inline long long rows_blocks(const TileCfg &t, int Lx, int Ly, int Lz)
{
    return (long long)rows_cut(Lx, t.cx / 64, -t.k).ntx * ((Ly + t.cy - 1) / t.cy) * ((Lz + t.cz - 1) / t.cz);
}

// One direction of a launch: n stencil levels (at most K), the first at bead `first`,
// forward upwards, backward downwards.
struct RowsHalf {
    int first, n;
    int start;     // the propagator starts here from the field factor (G_1, G+_N)
    int late;      // the bead's other visit was earlier: the slot holds its value, the term replaces it
    int from_pp;   // forward: the input is read from `in` (else from the slot of bead first - 1)
    int out;       // the last level is also written to `out`
};

struct RowsInfo {
    RowsHalf f, g;
    unsigned long long types;   // bit s - 1: species of bead s
    int N;
    int nf;                     // workgroups of the forward half
};

// Launch j (1 .. rows_launches) of the row sweeps for chains of N >= 2 beads: the N - 1
// stencil steps of a sweep are cut into m = ceil((N - 1) / K) nearly equal blocks of
// consecutive beads; launch j takes forward block j and backward block m + 1 + lag - j,
// lag = m mod 2, the schedule of the paired one-step sweeps with blocks for beads: a block's
// two visits never share a launch, the first leaves G_s or sigma[G+_{s+1}] in the slots and
// the second the term.  G_1 and G+_N are products of a field factor and start the first
// block of their sweep without a stencil.  Backward step 1 is left to the density launch.
struct RowsLaunch {
    RowsHalf f, g;
    bool has_f, has_g;
};
inline int rows_blocks_of(int N, int K) { return (N - 1 + K - 1) / K; }
inline int rows_launches(int N, int K)
{
    const int m = rows_blocks_of(N, K);
    return m + (m & 1);
}
inline RowsLaunch rows_schedule(int N, int K, int j)
{
    const int m = rows_blocks_of(N, K), lag = m & 1, se = (m + lag) / 2, bi = m + 1 + lag - j;
    // first bead of block i
    auto lo = [&](int i) {
        const int q = (N - 1) / m, r = (N - 1) % m;
        return 2 + (i - 1) * q + (i - 1 < r ? i - 1 : r);
    };
    RowsLaunch l{};
    l.has_f = j <= m;
    l.has_g = bi <= m;
    if (l.has_f) {
        l.f.first = lo(j);
        l.f.n = lo(j + 1) - lo(j);
        l.f.start = j == 1;
        l.f.late = j > se;
        l.f.from_pp = j >= 2 && j - 1 >= se;
        l.f.out = j >= se && j < m;
    }
    if (l.has_g) {
        const int hi = lo(bi + 1) - 1;
        l.g.start = hi == N;
        l.g.first = hi == N ? N - 1 : hi;
        l.g.n = l.g.first - lo(bi) + 1;
        l.g.late = bi <= se;
        l.g.out = 1;
    }
    return l;
}

template <typename real>
void launch_rows(const TileCfg &cfg, hipStream_t s, const Plan &p, const Rep *rep, RepState *st, const Chain &ch,
                 const RowsLaunch &l, PropBufs<real> b, const real *fin, real *fout,
                 const real *gin, real *gout, double *partG, int sums, hipEvent_t e0, hipEvent_t e1);

}  // namespace hsf
