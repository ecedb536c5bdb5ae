// prop_rows.h -- the row-resident paired sweeps (K contour steps per launch).
#pragma once

#include "prop_block.h"
#include "rows_schedule.h"

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

struct RowsInfo {
    RowsHalf f, g;
    unsigned long long types;   // bit s - 1: species of bead s
    int N;
    int nf;                     // workgroups of the forward half
};

template <typename real>
void launch_rows(const TileCfg &cfg, hipStream_t s, const Plan &p, const Rep *rep, RepState *st, const Chain &ch,
                 const RowsLaunch &l, PropBufs<real> b, const real *fin, real *fout,
                 const real *gin, real *gout, double *partG, int sums, hipEvent_t e0, hipEvent_t e1);

}  // namespace hsf
