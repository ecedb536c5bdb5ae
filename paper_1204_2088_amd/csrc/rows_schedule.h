// rows_schedule.h -- which steps the launches of the row-resident sweeps take (host code without
// device headers).
#pragma once

namespace hsf {

// One direction of a launch: n stencil levels (at most K), the first at bead `first`,
// forward upwards, backward downwards.
struct RowsHalf {
    int first, n;
    int start;     // the propagator starts here from the field factor (G_1, G+_N)
    int late;      // the bead's other visit was earlier: the slot holds its value, the term replaces it
    int from_pp;   // forward: the input is read from `in` (else from the slot of bead first - 1)
    int out;       // the last level is also written to `out`
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

// The forward sweep alone, every G_s into its slot (launches 1 .. rows_blocks_of): the one
// that measures the per-step scales.
inline RowsLaunch rows_forward(int N, int K, int j)
{
    RowsLaunch l = rows_schedule(N, K, j);
    l.has_g = false;
    l.f.late = l.f.from_pp = l.f.out = 0;
    return l;
}

}  // namespace hsf
