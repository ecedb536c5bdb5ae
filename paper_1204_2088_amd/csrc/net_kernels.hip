// net_kernels.hip -- kernels of the warm-start network: periodic 3x3x3
// convolutions as implicit GEMMs on the BF16 matrix cores (FP32 accumulation),
// the weight gradient as a second MFMA GEMM over sites, and the element-wise
// parts (activation, pooling, upsampling, skip sums, loss, Adam).
//
// Tensors are FP32 [batch][channel][site] with site = x + L (y + L z) on a
// periodic L^3 box.  A convolution layer's weights W[co][ci][k] (k = 9 (dz+1) +
// 3 (dy+1) + (dx+1)) are staged for the matrix cores as BF16 rows
// Wm[co][kk], kk = k * cip + ci (cip = ci rounded up to 8), zero beyond 27 cip
// and up to kp = a multiple of 32, and co padded to a multiple of 16.
//
// v_mfma_f32_16x16x32_bf16 lane layout (wave of 64): A (16 x 32): lane l holds
// row l % 16, k = 8 (l / 16) + j; B (32 x 16): column l % 16, same k; C (16 x 16):
// column l % 16, rows 4 (l / 16) + i.
#include <hip/hip_ext.h>
#include <algorithm>
#include <math.h>

#include <type_traits>

#include "device_common.h"
#include "net_internal.h"

namespace hsf {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int wrapL(int v, int L)
{
    v %= L;
    return v < 0 ? v + L : v;
}

__device__ __forceinline__ float silu(float y) { return y / (1.0f + __expf(-y)); }
// silu and its derivative for |y| < 80: the quotient by a reciprocal and one correction of the remainder (the
// scaling for overflow and underflow that a division adds is not needed there)
__device__ __forceinline__ float silu80(float y)
{
    const float d = 1.0f + __expf(-y), r = __builtin_amdgcn_rcpf(d), q = y * r;
    return __builtin_fmaf(__builtin_fmaf(-d, q, y), r, q);
}
__device__ __forceinline__ float silu_grad(float y)
{
    const float s = 1.0f / (1.0f + __expf(-y));
    return s * (1.0f + y * (1.0f - s));
}
__device__ __forceinline__ float silu_grad80(float y)
{
    const float d = 1.0f + __expf(-y), r = __builtin_amdgcn_rcpf(d);
    const float s = __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
    return s * (1.0f + y * (1.0f - s));
}

// Adds a contribution g to the gradient of element e of an activation; the last one turns the
// sum into the gradient of the pre-activation.
__device__ __forceinline__ void give_gradient(const ConvGive &t, long long e, float g)
{
    const float v = t.add ? t.dst[e] + g : g;
    t.dst[e] = t.Y ? v * silu_grad(t.Y[e]) : v;
}

// ---------------------------------------------------------------- forward convolution
// Y[b][co][x] = bias[co] + sum_{ci,k} W[co][ci][k] X[b][ci][x + off_k], written as
// ConvOut asks (pre-activation, FP32 activation, packed BF16 activation).  The input
// tile with a one-site halo is staged in LDS as BF16 16-byte units of 8 channels,
// unit-major: xs[cip / 8][halo site][8].  A B operand read takes one unit of 16
// consecutive sites, i.e. 16 consecutive units: no two lanes of a 16-lane group share
// an LDS bank, whatever cip is (site-major rows of cip >= 16 channels would put sites
// 8 apart on the same banks).  The weights follow in slabs of kSlab K chunks (32 rows
// of K each), [cop][kSlab * 32 + 8] (the 8 extra columns stagger the rows over the LDS
// banks), so the K loop reads only LDS; the next slab's loads are in flight while the
// current one is multiplied.  Small slabs keep a 16x8x4 block of a 16-channel layer
// under 40 KB of LDS, four blocks per CU.
// Bound by instructions around the products: a wave of a 64^3, batch 2, 16 -> 16 layer issues 1450
// vector instructions for 112 matrix ones, in the staging, the epilogue and their addresses
// (2170 with divisions by runtime counts, full divisions in SiLU and an address per store), and
// its LDS reads take a third of the 20.3 us (31.5 before).
constexpr int kSlab = 4;
constexpr int kSlabRow = kSlab * 32 + 8;

// Units of a plane of the staged tile (8 channels of every halo site), a multiple of 16: a 16-byte
// LDS read takes lanes of two 16-lane groups together (0-3 and 12-15 of one, 4-11 of the
// next), and with planes a multiple of 256 bytes apart those two groups, which read two planes
// at the same sites, share no bank (16x8x4 tile, 1080 units: 2.3M conflict cycles a launch,
// with 1088 0.5M).
template <int BX, int BY, int BZ>
constexpr int conv_plane()
{
    return ((BX + 2) * (BY + 2) * (BZ + 2) + 15) / 16 * 16;
}

// e / d for the small counts of a tile (0 <= e, e d < 2^16), e / D with a constant: one multiply
// and a shift.
__device__ __forceinline__ int div_small(int e, int inv) { return (int)(__umul24((unsigned)e, (unsigned)inv) >> 16); }
template <int D>
__device__ __forceinline__ int div_by(int e)
{
    return div_small(e, 65536 / D + 1);
}

// periodic index for -L <= v < 2L (boxes at least one tile wide), general otherwise
__device__ __forceinline__ int wrap_tile(int v, int L, bool small)
{
    if (small) return wrapL(v, L);
    return v < 0 ? v + L : (v >= L ? v - L : v);
}


// Value of input channel c of sample b at site (gx, gy, gz) of the convolution's
// L^3 box, read through the input's composition (ConvIn): the tensor itself, the sum
// of two tensors (decoder skip), the nearest 2x upsampling of a tensor on the
// (L/2)^3 box, or the 2x2x2 average of a tensor on the (2L)^3 box (summed in the
// order dz, dy, dx, as the pooling of the backward pass assumes).
__device__ __forceinline__ float conv_input(const ConvIn &in, int b, int c, int ci, int gx, int gy, int gz, int L)
{
    if (in.mode == CONV_IN_UP) {
        const int h = L >> 1;
        const long long vh = (long long)h * h * h;
        return in.x1[((long long)b * ci + c) * vh + (gx >> 1) + (long long)h * ((gy >> 1) + (long long)h * (gz >> 1))];
    }
    if (in.mode == CONV_IN_POOL) {
        const int f = L << 1;
        const long long vf = (long long)f * f * f;
        const float *p = in.x1 + ((long long)b * ci + c) * vf;
        float s = 0.0f;
        for (int dz = 0; dz < 2; ++dz)
            for (int dy = 0; dy < 2; ++dy)
                for (int dx = 0; dx < 2; ++dx)
                    s += p[(2 * gx + dx) + (long long)f * ((2 * gy + dy) + (long long)f * (2 * gz + dz))];
        return 0.125f * s;
    }
    const long long V = (long long)L * L * L;
    const long long e = ((long long)b * ci + c) * V + gx + (long long)L * (gy + (long long)L * gz);
    return in.mode == CONV_IN_ADD ? in.x1[e] + in.x2[e] : in.x1[e];
}

typedef float floatv4 __attribute__((ext_vector_type(4)));
typedef float floatv2 __attribute__((ext_vector_type(2)));

// The same in parts, for loops over channels: element conv_offset of a channel's data, channels
// conv_stride apart, is read for site (x, y, z); conv_load1 and conv_load4 (sites x .. x + 3 of a
// row, x and L multiples of 4, in wide loads) give the input's values from there.
template <int MODE>
__device__ __forceinline__ long long conv_stride(int L)
{
    const long long n = MODE == CONV_IN_UP ? L >> 1 : MODE == CONV_IN_POOL ? L << 1 : L;
    return n * n * n;
}
template <int MODE>
__device__ __forceinline__ long long conv_offset(int x, int y, int z, int L)
{
    if constexpr (MODE == CONV_IN_UP) return (x >> 1) + (long long)(L >> 1) * ((y >> 1) + (L >> 1) * (z >> 1));
    if constexpr (MODE == CONV_IN_POOL) return 2 * x + (long long)(L << 1) * (2 * y + (L << 1) * (2 * z));
    return x + (long long)L * (y + L * z);
}
template <int MODE>
__device__ __forceinline__ float conv_load1(const ConvIn &in, long long e, int L)
{
    if constexpr (MODE == CONV_IN_POOL) {
        const int f = L << 1;
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s += in.x1[e + (q & 1) + (long long)f * (((q >> 1) & 1) + (long long)f * (q >> 2))];
        return 0.125f * s;
    }
    return MODE == CONV_IN_ADD ? in.x1[e] + in.x2[e] : in.x1[e];
}
template <int MODE>
__device__ __forceinline__ floatv4 conv_load4(const ConvIn &in, long long e, int L)
{
    if constexpr (MODE == CONV_IN_UP) {
        const floatv2 v = *reinterpret_cast<const floatv2 *>(in.x1 + e);
        return floatv4{v.x, v.x, v.y, v.y};
    } else if constexpr (MODE == CONV_IN_POOL) {
        const int f = L << 1;
        floatv4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < 4; ++q) {   // (dz, dy) = (q / 2, q % 2)
            const float *r = in.x1 + e + ((long long)(q >> 1) * f + (q & 1)) * f;
            const floatv4 u = *reinterpret_cast<const floatv4 *>(r), v = *reinterpret_cast<const floatv4 *>(r + 4);
            s[0] = (s[0] + u[0]) + u[1];
            s[1] = (s[1] + u[2]) + u[3];
            s[2] = (s[2] + v[0]) + v[1];
            s[3] = (s[3] + v[2]) + v[3];
        }
        return 0.125f * s;
    } else {
        floatv4 v = *reinterpret_cast<const floatv4 *>(in.x1 + e);
        if constexpr (MODE == CONV_IN_ADD) v += *reinterpret_cast<const floatv4 *>(in.x2 + e);
        return v;
    }
}

// A BX x BY x BZ tile with its one-site halo, unit-major xs[cip / 8][h][8] (forward; planes conv_plane apart): a
// work item is one halo site and eight consecutive channels, written to LDS as one
// 16-byte unit; two items (16 loads) per thread are in flight at once.
template <int BX, int BY, int BZ>
__device__ __forceinline__ void stage_halo_sm(const ConvIn &in, int b, int ci, int cip, int L, int x0, int y0,
                                              int z0, __bf16 *xs)
{
    constexpr int GX = BX + 2, GY = BY + 2, GS = GX * GY * (BZ + 2);
    constexpr int BMAX = BX > BY ? (BX > BZ ? BX : BZ) : (BY > BZ ? BY : BZ);
    const bool small = L < BMAX;
    constexpr int GP = conv_plane<BX, BY, BZ>();
    const int oct = cip / 8, total = GS * oct;
    for (int e0 = threadIdx.x; e0 < total; e0 += 256 * 2) {
        float v[2][8];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = e0 + u * 256;
            const int c8 = e % oct, h = e / oct;
            const bool ok = e < total;
            const int hx = h % GX, hy = (h / GX) % GY, hz = h / (GX * GY);
            const int gx = wrap_tile(x0 + hx - 1, L, small), gy = wrap_tile(y0 + hy - 1, L, small),
                      gz = wrap_tile(z0 + hz - 1, L, small);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = c8 * 8 + j;
                v[u][j] = 0.0f;
                if (ok && c < ci) {
                    v[u][j] = conv_input(in, b, c, ci, gx, gy, gz, L);
                    if (in.shift) v[u][j] = (v[u][j] - in.shift[c]) * in.scale[c];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int e = e0 + u * 256;
            if (e < total) {
                bf16x8 pk;
#pragma unroll
                for (int j = 0; j < 8; ++j) pk[j] = (__bf16)v[u][j];
                *reinterpret_cast<bf16x8 *>(xs + ((e % oct) * GP + e / oct) * 8) = pk;
            }
        }
    }
}

// Row-vector staging of the same tile: four consecutive x sites per channel in aligned wide
// loads, on boxes at least a tile wide with L a multiple of 4 (three times fewer load
// instructions than one site per load; of an upsampled input 41 -> 32 us at 64^3, batch
// 2, 16 -> 8 channels; of a pooled one 21 -> 15 at 32^3, 8 -> 16).
template <int BX, int BY, int BZ, int MODE>
__device__ __forceinline__ void stage_halo_rows(const ConvIn &in, int b, int ci, int cip, int L, int x0, int y0,
                                                int z0, __bf16 *xs)
{
    constexpr int GX = BX + 2, GY = BY + 2, GZ = BZ + 2, GS = GX * GY * GZ;
    constexpr int NG = (BX + 8) / 4;   // float4 groups covering x in [x0 - 4, x0 + BX + 4)
    constexpr int U = MODE == CONV_IN_POOL ? 1 : 2;
    constexpr int GP = conv_plane<BX, BY, BZ>();
    static_assert(GY * GZ * NG * 4 * 4 < 65536 && GS * 18 < 65536, "div_small");
    const int oct = cip / 8, oinv = 65536 / oct + 1, total = GY * GZ * NG * oct;
    const long long stride = conv_stride<MODE>(L), base = (long long)b * ci * stride;
    for (int e0 = threadIdx.x; e0 < total; e0 += 256 * U) {
        floatv4 v[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * 256;
            const bool ok = e < total;
            const int r = div_small(e, oinv), c8 = e - r * oct;
            const int row = div_by<NG>(r), g = r - row * NG;
            const int hz = div_by<GY>(row), hy = row - hz * GY;
            int xb = x0 - 4 + 4 * g;   // a multiple of 4; wraps as a whole group
            xb = xb < 0 ? xb + L : (xb >= L ? xb - L : xb);
            const int gy = wrap_tile(y0 + hy - 1, L, false), gz = wrap_tile(z0 + hz - 1, L, false);
            const long long site = base + conv_offset<MODE>(xb, gy, gz, L);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int c = c8 * 8 + j;
                v[u][j] = floatv4{0.f, 0.f, 0.f, 0.f};
                if (ok && c < ci) {
                    v[u][j] = conv_load4<MODE>(in, site + c * stride, L);
                    if (in.shift) v[u][j] = (v[u][j] - in.shift[c]) * in.scale[c];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * 256;
            if (e < total) {
                const int r = div_small(e, oinv), c8 = e - r * oct;
                const int row = div_by<NG>(r), g = r - row * NG;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int hx = 4 * g + q - 3;   // halo x position of this site
                    if (hx >= 0 && hx < GX) {
                        bf16x8 pk;
#pragma unroll
                        for (int j = 0; j < 8; ++j) pk[j] = (__bf16)v[u][j][q];
                        *reinterpret_cast<bf16x8 *>(xs + (c8 * GP + row * GX + hx) * 8) = pk;
                    }
                }
            }
        }
    }
}

// The same tile from a packed BF16 input (CONV_IN_PACKED): halo unit e (site e / (cip /
// 8), channels 8 (e % (cip / 8)) + 0..7) is one 16-byte copy from global memory (site
// after site, so the loads are contiguous) to its unit-major LDS place; eight copies
// per thread are in flight at once.
template <int BX, int BY, int BZ>
__device__ __forceinline__ void stage_halo_packed(const __bf16 *__restrict__ xp, int b, int cip, int L, int x0,
                                                  int y0, int z0, __bf16 *xs)
{
    constexpr int GX = BX + 2, GY = BY + 2, GS = GX * GY * (BZ + 2);
    constexpr int BMAX = BX > BY ? (BX > BZ ? BX : BZ) : (BY > BZ ? BY : BZ);
    constexpr int U = 8;
    const bool small = L < BMAX;
    constexpr int GP = conv_plane<BX, BY, BZ>();
    const int oct = cip / 8, oinv = 65536 / oct + 1, total = GS * oct;
    static_assert(GS * 4 * 4 < 65536 && GS * GX < 65536, "div_small");
    const __bf16 *base = xp + (long long)b * L * L * L * cip;
    for (int e0 = threadIdx.x; e0 < total; e0 += 256 * U) {
        bf16x8 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * 256;
            if (e < total) {
                const int h = div_small(e, oinv), c8 = e - h * oct;
                const int row = div_by<GX>(h), hx = h - row * GX, hz = div_by<GY>(row), hy = row - hz * GY;
                const int gx = wrap_tile(x0 + hx - 1, L, small), gy = wrap_tile(y0 + hy - 1, L, small),
                          gz = wrap_tile(z0 + hz - 1, L, small);
                const unsigned long long site = (unsigned long long)((unsigned)gy + (unsigned)L * gz) * (unsigned)L + (unsigned)gx;
                v[u] = *reinterpret_cast<const bf16x8 *>(base + site * (unsigned)cip + 8 * c8);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = e0 + u * 256;
            const int h = div_small(e, oinv), c8 = e - h * oct;
            if (e < total) *reinterpret_cast<bf16x8 *>(xs + (c8 * GP + h) * 8) = v[u];
        }
    }
}

constexpr int kMaxKGroups = 27 * 32 / 8 + 4;   // K rows / 8 for cip <= 32, rounded up to 32 rows

template <int BX, int BY, int BZ>
constexpr size_t conv_fwd_lds_t(int cip, int cop)
{
    return (size_t)(conv_plane<BX, BY, BZ>() * cip + cop * kSlabRow) * sizeof(__bf16) +
           kMaxKGroups * sizeof(int);
}

// Block: a BX x BY x BZ tile of one sample; its 16-site MFMA column tiles are dealt to
// the four waves (NTW each), each with NM = cop / 16 (1 or 2) 16-channel output tiles.
// GIVE: the data gradient, which adds to ConvOut::give instead of writing Y, A or Ap (the sum and
// the derivative of the activation in the epilogue cost 2 us at 64^3, batch 2, 8 -> 8 channels,
// the passes over memory they replace 20).
// Four blocks of the 16-channel 16x8x4 tile per CU (LDS) need at most 128 registers.
template <int BX, int BY, int BZ, int NM, bool GIVE>
__global__ __launch_bounds__(256, BX == 16 && NM == 1 ? 4 : 1) void k_conv_fwd(ConvIn in, int ci, int cip, const __bf16 *__restrict__ Wm, int kp,
                                                   int co, int cop, const float *__restrict__ bias, ConvOut out, int L,
                                                   int tiles_x, int tiles_y, int tiles_per_sample)
{
    constexpr int BS = BX * BY * BZ, GX = BX + 2, GY = BY + 2, GP = conv_plane<BX, BY, BZ>();
    constexpr int NTW = BS / 64;   // column tiles per wave
    constexpr int NPRE = (NM * 16 * kSlab * 4 + 255) / 256;   // weight vectors per thread and slab
    static_assert(BS % 64 == 0 && BX % 8 == 0, "tile shape");
    extern __shared__ __align__(16) unsigned char smem[];
    __bf16 *xs = reinterpret_cast<__bf16 *>(smem);   // [cip / 8][GP][8]
    __bf16 *ws = xs + GP * cip;                       // [cop][kSlabRow]
    int *koff = reinterpret_cast<int *>(ws + cop * kSlabRow);   // [kp / 8]
    const int bid = plan_block();   // neighbouring tiles on one XCD
    const int b = bid / tiles_per_sample;
    int t = bid % tiles_per_sample;
    const int x0 = (t % tiles_x) * BX;
    t /= tiles_x;
    const int y0 = (t % tiles_y) * BY;
    const int z0 = (t / tiles_y) * BZ;
    const long long V = (long long)L * L * L;
    // weight slab k0 (rows of kp, k0 .. k0 + kSlab * 32) through registers: load(k0)
    // issues the loads, store(k0) writes what arrived to LDS
    bf16x8 wv[NPRE];
    auto slab_vectors = [&](int k0, int &vec_per_row) {
        vec_per_row = min(kSlab * 32, kp - k0) / 8;
        return cop * vec_per_row;
    };
    auto load_slab = [&](int k0) {
        int vpr;
        const int nvec = slab_vectors(k0, vpr);
#pragma unroll
        for (int u = 0; u < NPRE; ++u) {
            const int e = threadIdx.x + u * 256;
            if (e < nvec) {
                const int r = e / vpr, v8 = e - r * vpr;
                wv[u] = *reinterpret_cast<const bf16x8 *>(Wm + (long long)r * kp + k0 + 8 * v8);
            }
        }
    };
    auto store_slab = [&](int k0) {
        int vpr;
        const int nvec = slab_vectors(k0, vpr);
#pragma unroll
        for (int u = 0; u < NPRE; ++u) {
            const int e = threadIdx.x + u * 256;
            if (e < nvec) {
                const int r = e / vpr, v8 = e - r * vpr;
                *reinterpret_cast<bf16x8 *>(ws + r * kSlabRow + 8 * v8) = wv[u];
            }
        }
    };
    load_slab(0);   // in flight with the tile's loads
    // LDS element offset, relative to 8 times a site's halo position, of each group of
    // eight K rows (tap k, channels c0..c0+7: unit c0 / 8 of the tap's neighbour);
    // padding rows point at the centre tap (zero weights there)
    for (int g = threadIdx.x; g < kp / 8; g += 256) {
        int k = (8 * g) / cip;
        const int c0 = 8 * g - k * cip;
        if (k > 26) k = 13;
        koff[g] = ((((k / 9) - 1) * GX * GY + (((k / 3) % 3) - 1) * GX + ((k % 3) - 1)) + (c0 / 8) * GP) * 8;
    }
    if (in.mode == CONV_IN_PACKED)
        stage_halo_packed<BX, BY, BZ>(in.xp, b, cip, L, x0, y0, z0, xs);
    else if (L % 4 == 0 && L >= BX && L >= BY && L >= BZ) {
        switch (in.mode) {
        case CONV_IN_ADD: stage_halo_rows<BX, BY, BZ, CONV_IN_ADD>(in, b, ci, cip, L, x0, y0, z0, xs); break;
        case CONV_IN_UP: stage_halo_rows<BX, BY, BZ, CONV_IN_UP>(in, b, ci, cip, L, x0, y0, z0, xs); break;
        case CONV_IN_POOL: stage_halo_rows<BX, BY, BZ, CONV_IN_POOL>(in, b, ci, cip, L, x0, y0, z0, xs); break;
        default: stage_halo_rows<BX, BY, BZ, CONV_IN_PLAIN>(in, b, ci, cip, L, x0, y0, z0, xs);
        }
    }
    else
        stage_halo_sm<BX, BY, BZ>(in, b, ci, cip, L, x0, y0, z0, xs);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane >> 4, col = lane & 15;
    floatx4 acc[NTW][NM];
#pragma unroll
    for (int q = 0; q < NTW; ++q)
#pragma unroll
        for (int m = 0; m < NM; ++m) acc[q][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    // this lane's sites (column of the B operand): LDS element offsets of their halo
    // positions
    int hbase[NTW];
#pragma unroll
    for (int q = 0; q < NTW; ++q) {
        const int n = (wave * NTW + q) * 16 + col;
        const int tx = n % BX, ty = (n / BX) % BY, tz = n / (BX * BY);
        hbase[q] = ((tz + 1) * GX * GY + (ty + 1) * GX + (tx + 1)) * 8;
    }
    for (int k0 = 0; k0 < kp; k0 += kSlab * 32) {
        const int klen = min(kSlab * 32, kp - k0);
        __syncthreads();   // previous slab consumed (and, the first time, the halo staged)
        store_slab(k0);
        if (k0 + kSlab * 32 < kp) load_slab(k0 + kSlab * 32);
        __syncthreads();
        const __bf16 *wa = ws + col * kSlabRow + 8 * grp;
        const int *kg = koff + k0 / 8 + grp;
        for (int kc = 0; kc < klen; kc += 32) {
            const int off = kg[kc / 8];
            bf16x8 a[NM];
#pragma unroll
            for (int m = 0; m < NM; ++m) a[m] = *reinterpret_cast<const bf16x8 *>(wa + m * 16 * kSlabRow + kc);
#pragma unroll
            for (int q = 0; q < NTW; ++q) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(xs + hbase[q] + off);
#pragma unroll
                for (int m = 0; m < NM; ++m)
                    acc[q][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], bv, acc[q][m], 0, 0, 0);
            }
        }
    }
    if constexpr (GIVE) {   // a batch of sites' loads in flight before the first is needed
        constexpr int QB = NTW < 4 / NM ? NTW : 4 / NM;
        const long long first = ((long long)b * co + 4 * grp) * V;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const ConvGive to = out.give[d];
            if (!to.dst) continue;
#pragma unroll
            for (int q0 = 0; q0 < NTW; q0 += QB) {
                long long at[QB];
                float old[QB][NM][4], pre[QB][NM][4], top = 0.0f;
#pragma unroll
                for (int q = 0; q < QB; ++q) {
                    const int n = (wave * NTW + q0 + q) * 16 + col;
                    const int gx = x0 + n % BX, gy = y0 + (n / BX) % BY, gz = z0 + n / (BX * BY);
                    at[q] = gx < L && gy < L && gz < L
                                ? (long long)((unsigned long long)((unsigned)gy + (unsigned)L * gz) * (unsigned)L + (unsigned)gx)
                                : -1;
                }
#pragma unroll
                for (int q = 0; q < QB; ++q)
#pragma unroll
                    for (int m = 0; m < NM; ++m)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            old[q][m][i] = pre[q][m][i] = 0.0f;
                            if (at[q] >= 0 && m * 16 + 4 * grp + i < co) {
                                if (to.add) old[q][m][i] = to.dst[first + (m * 16 + i) * V + at[q]];
                                if (to.Y) pre[q][m][i] = to.Y[first + (m * 16 + i) * V + at[q]];
                            }
                            top = fmaxf(top, fabsf(pre[q][m][i]));
                        }
                auto write = [&](auto grad) {
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int m = 0; m < NM; ++m)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                float v = acc[q0 + q][m][i];
                                if (to.add) v = old[q][m][i] + v;
                                if (to.Y) v *= grad(pre[q][m][i]);
                                if (at[q] >= 0 && m * 16 + 4 * grp + i < co)
                                    to.dst[first + (m * 16 + i) * V + at[q]] = v;
                            }
                };
                if (__ballot(!(top < 80.0f)) == 0) write([](float y) { return silu_grad80(y); });
                else write([](float y) { return silu_grad(y); });
            }
        }
        return;
    }
    // epilogue: lane holds rows 4 grp + i of each M tile, column = its site
    float bo[NM][4], top = 0.0f;
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int o = m * 16 + 4 * grp + i;
            bo[m][i] = bias && o < co ? bias[o] : 0.0f;
        }
#pragma unroll
    for (int q = 0; q < NTW; ++q)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[q][m][i] += bo[m][i];
                top = fmaxf(top, fabsf(acc[q][m][i]));
            }
    const int cpk = (co + 7) & ~7;   // channel stride of the packed activation
    __bf16 *Pb = out.Ap ? out.Ap + (long long)b * V * cpk + 4 * grp : nullptr;
    const long long first = ((long long)b * co + 4 * grp) * V;
    float *Yb = out.Y ? out.Y + first : nullptr, *Ab = out.A ? out.A + first : nullptr;
    auto write = [&](auto act) {
#pragma unroll
        for (int q = 0; q < NTW; ++q) {
            const int n = (wave * NTW + q) * 16 + col;
            const int gx = x0 + n % BX, gy = y0 + (n / BX) % BY, gz = z0 + n / (BX * BY);
            if (gx >= L || gy >= L || gz >= L) continue;
            const unsigned long long site = (unsigned long long)((unsigned)gy + (unsigned)L * gz) * (unsigned)L + (unsigned)gx;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int o0 = m * 16 + 4 * grp;
                floatx4 a = acc[q][m];
                if (Pb || Ab) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[i] = act(a[i]);
                }
                if (Pb && o0 < cpk) {   // four consecutive channels of the site: one 8-byte store
                    bf16x4 pk;
#pragma unroll
                    for (int i = 0; i < 4; ++i) pk[i] = (__bf16)(o0 + i < co ? a[i] : 0.0f);
                    *reinterpret_cast<bf16x4 *>(Pb + site * (unsigned)cpk + m * 16) = pk;
                }
                if (Yb || Ab) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (o0 + i >= co) continue;
                        if (Ab) Ab[(m * 16 + i) * V + site] = a[i];
                        float y = acc[q][m][i];
                        if (out.shift) y = (y - out.shift[o0 + i]) * out.scale[o0 + i];
                        if (Yb) Yb[(m * 16 + i) * V + site] = y;
                    }
                }
            }
        }
    };
    // infinities and large values, which silu80 does not take, are rare: one test per wave
    if (__ballot(!(top < 80.0f)) == 0) write([](float y) { return silu80(y); });
    else write([](float y) { return silu(y); });
}

// ---------------------------------------------------------------- weight gradient
// dW[o][c][k] = sum_b sum_x dY[b][o][x] X[b][c][x + off_k], a contraction over the sites, for the
// layers of one box in one launch (on coarse levels a layer alone has a few blocks).  Block
// (layer, g, sl) owns the input channels 8 g .. 8 g + 7 and the site tiles sl, sl + slices, ...
// of 8 XC x 4 x 4 sites.  Its C matrix is (output channels) x (9 row offsets (dz, dy) x 8
// channels) for each dx: 5 column tiles of 16 and 3 dx, in registers, once per wave; the four
// waves take the 32-site K chunks in turn and their sums are added at the end.  The B operand
// for dx = 0 (8 sites of a row) is one aligned LDS read, those for dx = -1 and +1 are funnel
// shifts of it with a neighbouring word, so an input site is staged once (16-byte loads, 8-byte
// LDS stores).  The A operand (8 sites of dY) goes from memory to registers: with the channels
// split over blocks no other wave of the block needs it.  The bias gradient is summed (FP64)
// from the same values.
//
// Bound by staging: the latency of its loads and a barrier pair per tile (60 matrix
// instructions per wave).  Measured at 64^3, batch 2 (8 -> 8 channels alone): 18 us, of which
// the 34 MB of X and dY take 7 at the rate of a copy; three x-shifted LDS copies staged value by
// value, a launch per layer, took 82.  The five layers of that level together 80 us against
// 501, four layers of 32^3 (16 channels) 32 against 134, of 16^3 (24) 22 against 125, two of 8^3
// (32) 13 against 67.
constexpr int kWgTY = 4, kWgTZ = 4, kWgRows = (kWgTY + 2) * (kWgTZ + 2);
constexpr int kWgCols = 5;             // 16-column tiles of 9 x 8 columns
constexpr int kWgElems = 27 * 8;       // weights of one output channel in a block

// LDS places: row r of channel c at wg_at(c, r): sites x0 .. x0 + XW - 1, then x0 + XW; x0 - 1 just
// before it.
template <int XC>
struct WgTile {
    static constexpr int XW = 8 * XC, PITCH = XW + 8, CP = kWgRows * PITCH + 8, LEAD = 8, SIZE = LEAD + 8 * CP;
    static __device__ __forceinline__ int at(int c, int row) { return LEAD + c * CP + row * PITCH; }
};

// Channels 8 g .. 8 g + 7 of a tile's rows.
template <int MODE, bool VEC, int XC>
__device__ __forceinline__ void wgrad_stage(const ConvIn &in, int ci, int b, int g, int x0, int y0, int z0, int L,
                                            __bf16 *xs)
{
    using T = WgTile<XC>;
    const int wave = threadIdx.x >> 6;
            // groups of four sites: of the first 32 rows a thread takes one place and 2 XC channels, of
            // the last 4 one place and channel; then the rows' two neighbours
            const long long stride = conv_stride<MODE>(L), base = ((long long)b * ci + 8 * g) * stride;
            auto wrap = [&](int v) {
                if constexpr (!VEC) return wrapL(v, L);
                v = v < 0 ? v + L : v;   // -L <= v < 3 L
                v = v >= L ? v - L : v;
                return v >= L ? v - L : v;
            };
            auto place = [&](int row, int x) {
                return base + conv_offset<MODE>(wrap(x0 + x), wrap(y0 + row % (kWgTY + 2) - 1),
                                                wrap(z0 + row / (kWgTY + 2) - 1), L);
            };
            auto group = [&](long long e, int row, int q) {
                if constexpr (VEC) return conv_load4<MODE>(in, e, L);
                floatv4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = conv_load1<MODE>(in, e - place(row, 4 * q) + place(row, 4 * q + i), L);
                return v;
            };
            auto store = [&](int c, int row, int q, const floatv4 &v) {
                bf16x4 w;
#pragma unroll
                for (int i = 0; i < 4; ++i) w[i] = (__bf16)v[i];
                *reinterpret_cast<bf16x4 *>(xs + T::at(c, row) + 4 * q) = w;
            };
            int tid = threadIdx.x;   // opaque: places are computed per tile, not kept in registers
            asm volatile("" : "+v"(tid));
            {
                constexpr int NC = 2 * XC, U = MODE == CONV_IN_POOL ? 1 : MODE == CONV_IN_ADD ? (NC < 4 ? NC : 4) : NC;
                const int p = tid % (64 * XC), row = p / (2 * XC), q = p % (2 * XC), c0 = wave / XC * NC;
                const long long e = place(row, 4 * q) + c0 * stride;
#pragma unroll
                for (int i0 = 0; i0 < NC; i0 += U) {
                    floatv4 v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        v[u] = floatv4{0.f, 0.f, 0.f, 0.f};
                        if (8 * g + c0 + i0 + u < ci) v[u] = group(e + (i0 + u) * stride, row, q);
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) store(c0 + i0 + u, row, q, v[u]);
                }
            }
            if (tid < 64 * XC) {
                const int p = tid % (8 * XC), row = 32 + p / (2 * XC), q = p % (2 * XC), c = tid / (8 * XC);
                floatv4 v = {0.f, 0.f, 0.f, 0.f};
                if (8 * g + c < ci) v = group(place(row, 4 * q) + c * stride, row, q);
                store(c, row, q, v);
            }
            if (tid < 6 * kWgRows) {
                const int p = tid % (2 * kWgRows), row = p >> 1, x = (p & 1) ? T::XW : -1, c0 = tid / (2 * kWgRows);
                const long long e = place(row, x);
                float v[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int c = c0 + 3 * i;
                    v[i] = 0.0f;
                    if (c < 8 && 8 * g + c < ci) v[i] = conv_load1<MODE>(in, e + c * stride, L);
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    if (c0 + 3 * i < 8) xs[T::at(c0 + 3 * i, row) + x] = (__bf16)v[i];
            }
}

// VEC: L is a multiple of 4 and rows are read in 16-byte loads.
template <bool VEC, int XC, int MT>
__global__ __launch_bounds__(256, MT == 1 ? 3 : 2) void k_conv_wgrad(WgradJobs W, int L, int tiles_x,
                                                                                     int tiles_y, int tiles_per_sample,
                                                                                     int n_tiles)
{
    using T = WgTile<XC>;
    constexpr int XW = T::XW, PITCH = T::PITCH;
    constexpr size_t kX = sizeof(__bf16) * T::SIZE, kR = sizeof(floatx4) * 2 * kWgCols * 64;
    __shared__ __align__(16) unsigned char smem[kX > kR ? kX : kR];   // the tile; then the waves' sums
    __shared__ double bs[16][MT * 16];
    __bf16 *xs = reinterpret_cast<__bf16 *>(smem);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, grp = lane >> 4, col = lane & 15;
    // the last layer that starts at or before this block
    const int job = __builtin_popcountll(__ballot(lane < W.n && W.j[min(lane, W.n - 1)].block0 <= (int)blockIdx.x)) - 1;
    const WgradJob J = W.j[job];
    const int slices = J.slices, co = J.co;
    const int g = ((int)blockIdx.x - J.block0) / slices, sl = ((int)blockIdx.x - J.block0) % slices;
    const float *dY = J.dY;
    const long long V = (long long)L * L * L;
    int boff[kWgCols];
#pragma unroll
    for (int t = 0; t < kWgCols; ++t) {
        const int j = t * 16 + col, r = min(j >> 3, 8);   // columns beyond 72 are dropped
        boff[t] = T::at(j & 7, (r / 3) * (kWgTY + 2) + r % 3);
    }
    floatx4 acc[MT][kWgCols][3];
    double bsum[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        bsum[m] = 0.0;
#pragma unroll
        for (int t = 0; t < kWgCols; ++t)
#pragma unroll
            for (int d = 0; d < 3; ++d) acc[m][t][d] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    for (int tile = sl; tile < n_tiles; tile += slices) {
        const int b = tile / tiles_per_sample;
        int t = tile % tiles_per_sample;
        const int x0 = (t % tiles_x) * XW;
        t /= tiles_x;
        const int y0 = (t % tiles_y) * kWgTY, z0 = (t / tiles_y) * kWgTZ;
        // this wave's A operands: chunk wave + 4 j holds the 8-site groups 4 (wave + 4 j) + grp;
        // the next chunk's loads are in flight while one is multiplied
        float a[2][MT][8];
        auto load_a = [&](int j, float (&v)[MT][8]) {
            const int q = 4 * (wave + 4 * j) + grp, row = q / XC;
            const int gx = x0 + 8 * (q % XC), gy = y0 + (row & 3), gz = z0 + (row >> 2);
            const bool in_box = gy < L && gz < L;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int o = m * 16 + col;
                const float *p = dY + ((long long)b * co + o) * V + ((long long)gz * L + gy) * L + gx;
                if constexpr (VEC) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        floatv4 w = {0.f, 0.f, 0.f, 0.f};
                        if (in_box && o < co && gx + 4 * h < L) w = *reinterpret_cast<const floatv4 *>(p + 4 * h);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[m][4 * h + i] = w[i];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[m][i] = in_box && o < co && gx + i < L ? p[i] : 0.0f;
                }
            }
        };
        load_a(0, a[0]);
        __syncthreads();   // the previous tile has been read
        switch (J.in.mode) {
        case CONV_IN_ADD: wgrad_stage<CONV_IN_ADD, VEC, XC>(J.in, J.ci, b, g, x0, y0, z0, L, xs); break;
        case CONV_IN_UP: wgrad_stage<CONV_IN_UP, VEC, XC>(J.in, J.ci, b, g, x0, y0, z0, L, xs); break;
        case CONV_IN_POOL: wgrad_stage<CONV_IN_POOL, VEC, XC>(J.in, J.ci, b, g, x0, y0, z0, L, xs); break;
        default: wgrad_stage<CONV_IN_PLAIN, VEC, XC>(J.in, J.ci, b, g, x0, y0, z0, L, xs);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < XC; ++j) {
            if (j + 1 < XC) load_a(j + 1, a[(j + 1) & 1]);
            bf16x8 ab[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    ab[m][i] = (__bf16)a[j & 1][m][i];
                    bsum[m] += (double)a[j & 1][m][i];
                }
            const int q = 4 * (wave + 4 * j) + grp, row = q / XC;
            const int roff = ((row >> 2) * (kWgTY + 2) + (row & 3)) * PITCH + 8 * (q % XC);
#pragma unroll
            for (int t = 0; t < kWgCols; ++t) {
                const __bf16 *p = xs + boff[t] + roff;
                const uint4 w = *reinterpret_cast<const uint4 *>(p);
                const unsigned lo = *reinterpret_cast<const unsigned *>(p - 2);
                const unsigned hi = *reinterpret_cast<const unsigned *>(p + 8);
                const unsigned s1 = __builtin_amdgcn_alignbit(w.y, w.x, 16), s2 = __builtin_amdgcn_alignbit(w.z, w.y, 16),
                               s3 = __builtin_amdgcn_alignbit(w.w, w.z, 16);
                const uint4 bl = {__builtin_amdgcn_alignbit(w.x, lo, 16), s1, s2, s3};
                const uint4 br = {s1, s2, s3, __builtin_amdgcn_alignbit(hi, w.w, 16)};
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    acc[m][t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab[m], __builtin_bit_cast(bf16x8, bl),
                                                                           acc[m][t][0], 0, 0, 0);
                    acc[m][t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab[m], __builtin_bit_cast(bf16x8, w),
                                                                           acc[m][t][1], 0, 0, 0);
                    acc[m][t][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ab[m], __builtin_bit_cast(bf16x8, br),
                                                                           acc[m][t][2], 0, 0, 0);
                }
            }
        }
    }
    // the waves' sums, (0 + 2) + (1 + 3), and the result of wave 0 to the slice's partials
    floatx4 *red = reinterpret_cast<floatx4 *>(smem);
    float *P = J.part + ((long long)g * slices + sl) * co * kWgElems;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
#pragma unroll
            for (int half = 2; half > 0; half >>= 1) {
                __syncthreads();
                if (wave >= half && wave < 2 * half)
#pragma unroll
                    for (int t = 0; t < kWgCols; ++t) red[((wave - half) * kWgCols + t) * 64 + lane] = acc[m][t][d];
                __syncthreads();
                if (wave < half)
#pragma unroll
                    for (int t = 0; t < kWgCols; ++t) acc[m][t][d] += red[(wave * kWgCols + t) * 64 + lane];
            }
            if (wave == 0)
#pragma unroll
                for (int t = 0; t < kWgCols; ++t) {
                    const int j = t * 16 + col;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int o = m * 16 + 4 * grp + i;
                        if (o < co && j < 72) P[o * kWgElems + ((j >> 3) * 3 + d) * 8 + (j & 7)] = acc[m][t][d][i];
                    }
                }
        }
    if (g > 0) return;
#pragma unroll
    for (int m = 0; m < MT; ++m) bs[wave * 4 + grp][m * 16 + col] = bsum[m];
    __syncthreads();
    if ((int)threadIdx.x < co) {
        double t = 0.0;
        for (int j = 0; j < 16; ++j) t += bs[j][threadIdx.x];
        J.bpart[(long long)sl * co + threadIdx.x] = t;
    }
}

// Sums of all layers' partials over their slices, in a fixed order, into the parameter vector's
// layout.  A block takes 32 consecutive elements of one layer, 32 threads for each four (slices
// j, j + 32, ... and then the 32 sums in order); a layer's last block its bias.  Bound by the
// latency of two batches of eight loads: 14 us for the 15 layers of a four-level network (a launch
// per layer for the sums, the reordering, and two for the bias took 370).
__global__ __launch_bounds__(256) void k_wgrad_sum(WgradSums W, const float *__restrict__ part,
                                                   const double *__restrict__ bpart, float *__restrict__ grad)
{
    __shared__ __align__(16) float red[4 * 256];
    double *redd = reinterpret_cast<double *>(red);
    const int lane = threadIdx.x & 63;   // the last layer that starts at or before this block
    const int l = __builtin_popcountll(__ballot(lane < W.n && W.l[min(lane, W.n - 1)].block0 <= (int)blockIdx.x)) - 1;
    const WgradSum S = W.l[l];
    const int blk = (int)blockIdx.x - S.block0, per = S.co * kWgElems, n = (S.ci + 7) / 8 * per;
    if (blk * 32 < n) {
        floatx4 *red4 = reinterpret_cast<floatx4 *>(red);
        const int j = threadIdx.x >> 3, e = blk * 32 + 4 * (threadIdx.x & 7);   // 4 divides per
        const int g = e / per, r = e % per;
        floatx4 s = {0.f, 0.f, 0.f, 0.f};
        if (e < n) {
            const floatx4 *p = reinterpret_cast<const floatx4 *>(part + S.part + (long long)g * S.slices * per + r);
            const long long step = per / 4;
            int k = j;
            for (; k + 7 * 32 < S.slices; k += 8 * 32) {
                floatx4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = p[(k + u * 32) * step];
#pragma unroll
                for (int u = 0; u < 8; ++u) s += v[u];
            }
            for (; k < S.slices; k += 32) s += p[k * step];
        }
        red4[threadIdx.x] = s;
        __syncthreads();
        if (j == 0 && e < n) {
            floatx4 t = red4[threadIdx.x];
#pragma unroll
            for (int q = 1; q < 32; ++q) t += red4[q * 8 + threadIdx.x];
            const int o = r / kWgElems, k = r % kWgElems;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = 8 * g + (k & 7) + i;
                if (c < S.ci) grad[S.w_off + ((long long)o * S.ci + c) * 27 + (k >> 3)] = t[i];
            }
        }
        return;
    }
    const int o = threadIdx.x & 31, j = threadIdx.x >> 5;
    double s = 0.0;
    if (o < S.co)
        for (int k = j; k < S.slices; k += 8) s += bpart[S.bpart + (long long)k * S.co + o];
    redd[threadIdx.x] = s;
    __syncthreads();
    if (j == 0 && o < S.co) {
        double t = redd[threadIdx.x];
        for (int q = 1; q < 8; ++q) t += redd[q * 32 + threadIdx.x];
        grad[S.b_off + o] = (float)t;
    }
}

// ---------------------------------------------------------------- element-wise parts
// gradient of the pooling: a fine site is given dout[coarse] / 8.  A thread takes two sites of a
// row (L is even).
__global__ void k_pool_bwd(const float *__restrict__ dout, ConvGive to, int L, long long n_in)
{
    const long long e = 2 * ((long long)blockIdx.x * blockDim.x + threadIdx.x);
    if (e >= n_in) return;
    const int h = L / 2, x = (int)(e % L);
    const long long row = e / L, yz = row % ((long long)L * L), bc = row / ((long long)L * L);
    const int y = (int)(yz % L), z = (int)(yz / L);
    const float g = 0.125f * dout[bc * h * h * h + x / 2 + (long long)h * (y / 2 + (long long)h * (z / 2))];
    floatv2 v = {g, g};
    if (to.add) v = *reinterpret_cast<const floatv2 *>(to.dst + e) + g;
    if (to.Y) {
        const floatv2 p = *reinterpret_cast<const floatv2 *>(to.Y + e);
        v = floatv2{v.x * silu_grad(p.x), v.y * silu_grad(p.y)};
    }
    *reinterpret_cast<floatv2 *>(to.dst + e) = v;
}

// gradient of the upsampling: a coarse site is given the sum of its 8 fine gradients
__global__ void k_up_bwd(const float *__restrict__ dout, ConvGive to, int L, long long n_in)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n_in) return;
    const int h = L / 2;
    const long long vo = (long long)L * L * L, vi = (long long)h * h * h;
    const long long bc = e / vi, r = e % vi;
    const int x = (int)(r % h), y = (int)((r / h) % h), z = (int)(r / ((long long)h * h));
    const float *p = dout + bc * vo;
    float s = 0.0f;
    for (int dz = 0; dz < 2; ++dz)
        for (int dy = 0; dy < 2; ++dy)
            for (int dx = 0; dx < 2; ++dx) s += p[(2 * x + dx) + (long long)L * ((2 * y + dy) + (long long)L * (2 * z + dz))];
    give_gradient(to, e, s);
}

// squared error: per-block partial sums of (p - t)^2 and dp = 2 (p - t) / count
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ p, const float *__restrict__ t,
                                             float *__restrict__ dp, long long n, float inv_count,
                                             double *__restrict__ part)
{
    const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
    double v = 0.0;
    if (e < n) {
        const float d = p[e] - t[e];
        v = (double)d * d;
        if (dp) dp[e] = 2.0f * d * inv_count;
    }
    __shared__ double red[256];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Adam step on the FP32 master parameters.
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, long long n, float lr, float b1, float b2, float eps, float c1,
                       float c2)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const float ge = g[e];
    const float me = b1 * m[e] + (1.0f - b1) * ge;
    const float ve = b2 * v[e] + (1.0f - b2) * ge * ge;
    m[e] = me;
    v[e] = ve;
    w[e] -= lr * (me / c1) / (sqrtf(ve / c2) + eps);
}

// BF16 matrix-core rows of one layer from its FP32 weights W[co][ci][27]:
//   fwd: Wm[o][k cip + c] = W[o][c][k]
//   dgrad (transposed, flipped): Wt[c][k cop' + o] = W[o][c][26 - k]  (cop' = co rounded up to 8)
__global__ void k_stage_weights(const float *__restrict__ W, int co, int ci, int cip, int kp, int cop_rows,
                                __bf16 *__restrict__ Wm, int cip_t, int kp_t, int cop_rows_t,
                                __bf16 *__restrict__ Wt)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long nf = (long long)cop_rows * kp, nt = (long long)cop_rows_t * kp_t;
    if (e < nf) {
        const int o = (int)(e / kp), kk = (int)(e % kp);
        const int k = kk / cip, c = kk % cip;
        float v = 0.0f;
        if (o < co && k < 27 && c < ci) v = W[((long long)o * ci + c) * 27 + k];
        Wm[e] = (__bf16)v;
    } else if (e < nf + nt) {
        const long long f = e - nf;
        const int c = (int)(f / kp_t), kk = (int)(f % kp_t);
        const int k = kk / cip_t, o = kk % cip_t;
        float v = 0.0f;
        if (c < ci && k < 27 && o < co) v = W[((long long)o * ci + c) * 27 + (26 - k)];
        Wt[f] = (__bf16)v;
    }
}

// Warm start from the network's prediction p (FP32, 2 polymer channels):
//   mode 0: w_I = p_I;  mode 1: w_I += p_I - p_prev_I
// ---------------------------------------------------------------- warm start
// Difference of densities used as the network's second input group:
//   mode 1: delta = phi - h0                (first difference)
//   mode 2: delta = phi - 2 h0 + h1         (second difference)
__device__ __forceinline__ double warm_delta(const double *phi, const double *h0, const double *h1, long long e,
                                             int mode)
{
    return mode == 2 ? (phi[e] - 2.0 * h0[e] + h1[e]) : (phi[e] - h0[e]);
}

// Per-block partial sums of delta^2 over the nsp x V values of one replica.
__global__ __launch_bounds__(256) void k_delta_sumsq(const double *__restrict__ phi, const double *__restrict__ h0,
                                                     const double *__restrict__ h1, long long n, int mode,
                                                     double *__restrict__ part)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long long)gridDim.x * 256) {
        const double d = warm_delta(phi, h0, h1, e, mode);
        acc += d * d;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// rms = sqrt(sum of the partials / n), floored so that a zero difference divides safely.
__global__ __launch_bounds__(256) void k_delta_rms(const double *__restrict__ part, int nparts, long long n,
                                                   double *__restrict__ rms)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < nparts; i += 256) acc += part[i];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) rms[0] = fmax(sqrt(red[0] / (double)n), 1e-300);
}

// Network input of one replica ([channel][V] FP32):
//   mode 0: x = phi                                   (nsp channels)
//   mode 1, 2: x = (h0, delta / rms)                  (2 nsp channels)
__global__ void k_net_input(const double *__restrict__ phi, const double *__restrict__ h0,
                            const double *__restrict__ h1, long long n, int mode, const double *__restrict__ rms,
                            float *__restrict__ x)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    if (mode == 0) {
        x[e] = (float)phi[e];
        return;
    }
    x[e] = (float)h0[e];
    x[n + e] = (float)(warm_delta(phi, h0, h1, e, mode) / rms[0]);
}

// Apply the prediction p ([2][V]) to the polymer fields w ([2][V] of the replica):
//   mode 0: w = p;  mode 1: w += rms p;  mode 2: w += (wh0 - wh1) + rms p.
__global__ void k_warm_apply(double *__restrict__ w, const float *__restrict__ p, long long n, int mode,
                             const double *__restrict__ rms, const double *__restrict__ wh0,
                             const double *__restrict__ wh1)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    if (mode == 0) {
        w[e] = (double)p[e];
        return;
    }
    double v = w[e] + rms[0] * (double)p[e];
    if (mode == 2) v += wh0[e] - wh1[e];
    w[e] = v;
}

// Training target of one replica over the polymer channels (the first 2 V values of the
// field layout): mode 0, the fields themselves; modes 1 and 2, delta w / rms with delta as
// in warm_delta.
__global__ void k_net_target(const double *__restrict__ w, const double *__restrict__ w0,
                             const double *__restrict__ w1, long long n, int mode, const double *__restrict__ rms,
                             float *__restrict__ y)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) y[e] = (float)(mode == 0 ? w[e] : warm_delta(w, w0, w1, e, mode) / rms[0]);
}

// Per-channel partial sums of x and x^2 over batch and sites: block (c, k) of a grid of
// C x nblk blocks covers every nblk-th chunk of 256 values of channel c.
__global__ __launch_bounds__(256) void k_channel_sums(const float *__restrict__ x, int batch, int C, long long V,
                                                      int nblk, double *__restrict__ part)
{
    const int c = blockIdx.x, k = blockIdx.y;
    __shared__ double r1[256], r2[256];
    double s1 = 0.0, s2 = 0.0;
    const long long n = (long long)batch * V;
    for (long long e = (long long)k * 256 + threadIdx.x; e < n; e += (long long)nblk * 256) {
        const long long b = e / V, i = e - b * V;
        const double v = (double)x[(b * C + c) * V + i];
        s1 += v;
        s2 += v * v;
    }
    r1[threadIdx.x] = s1;
    r2[threadIdx.x] = s2;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (threadIdx.x < h) {
            r1[threadIdx.x] += r1[threadIdx.x + h];
            r2[threadIdx.x] += r2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * ((long long)c * nblk + k)] = r1[0];
        part[2 * ((long long)c * nblk + k) + 1] = r2[0];
    }
}

// out[2 c] = mean, out[2 c + 1] = root mean square of channel c (partials summed in order).
__global__ void k_channel_finish(const double *__restrict__ part, int C, int nblk, double count,
                                 double *__restrict__ out)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    double s1 = 0.0, s2 = 0.0;
    for (int k = 0; k < nblk; ++k) {
        s1 += part[2 * ((long long)c * nblk + k)];
        s2 += part[2 * ((long long)c * nblk + k) + 1];
    }
    out[2 * c] = s1 / count;
    out[2 * c + 1] = sqrt(s2 / count);
}

// w += wh0 - wh1 (plain extrapolation of the fields)
__global__ void k_shift_fields(double *__restrict__ w, const double *__restrict__ wh0,
                               const double *__restrict__ wh1, long long n)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < n) w[e] += wh0[e] - wh1[e];
}

// x[b][c][v] = (x - shift[c]) * scale[c]  (input normalisation of the network)
__global__ void k_affine(float *__restrict__ x, int C, long long V, long long n, const float *__restrict__ shift,
                         const float *__restrict__ scale)
{
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int c = (int)((e / V) % C);
    x[e] = (x[e] - shift[c]) * scale[c];
}


// ---------------------------------------------------------------- launchers
static inline unsigned nb(long long n, int t) { return (unsigned)((n + t - 1) / t); }

// Largest dynamic LDS a block may use on the current device (queried once).
static size_t lds_limit()
{
    static size_t lim = 0;
    if (!lim) {
        int dev = 0, v = 0;
        lim = 65536;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess && v > 0)
            lim = std::min<size_t>((size_t)v, 65536);
    }
    return lim;
}

template <int BX, int BY, int BZ>
static void conv_fwd_launch(hipStream_t s, ConvIn in, int B, int ci, int cip, const __bf16 *Wm, int kp, int co,
                            int cop, const float *bias, ConvOut out, int L)
{
    const int tx = (L + BX - 1) / BX, ty = (L + BY - 1) / BY, tz = (L + BZ - 1) / BZ;
    const int tps = tx * ty * tz;
    const size_t lds = conv_fwd_lds_t<BX, BY, BZ>(cip, cop);
    auto go = [&](auto NM, auto GIVE) {
        hipLaunchKernelGGL((k_conv_fwd<BX, BY, BZ, NM(), GIVE()>), dim3(B * tps), dim3(256), lds, s, in, ci, cip, Wm, kp,
                           co, cop, bias, out, L, tx, ty, tps);
    };
    auto tiles = [&](auto GIVE) {
        if (cop == 16) go(std::integral_constant<int, 1>(), GIVE);
        else go(std::integral_constant<int, 2>(), GIVE);
    };
    if (out.give[0].dst) tiles(std::true_type());
    else tiles(std::false_type());
}

// Tile per layer: the largest of 16x8x4, 8x8x4, 8x4x4 that the box fills, whose LDS
// (halo tile plus one weight slab) fits, and that still gives the launch at least
// kMinConvBlocks blocks; else 8x4x2.  Larger tiles re-read fewer halo sites and stage
// the weights for more sites; on the coarse levels of a U-Net (8^3, 16^3 boxes) they
// would leave a launch with a handful of blocks, each working through all of its sites
// in turn.  The tile does not change any result: every output sums its K chunks in the
// same order.
constexpr long long kMinConvBlocks = 256;

static long long conv_blocks(int B, int L, int bx, int by, int bz)
{
    return (long long)B * ((L + bx - 1) / bx) * ((L + by - 1) / by) * ((L + bz - 1) / bz);
}

void net_conv_fwd(hipStream_t s, ConvIn in, int B, int ci, int cip, const __bf16 *Wm, int kp, int co, int cop,
                  const float *bias, ConvOut out, int L)
{
    const size_t lim = lds_limit();
    if (L >= 16 && conv_fwd_lds_t<16, 8, 4>(cip, cop) <= lim && conv_blocks(B, L, 16, 8, 4) >= kMinConvBlocks)
        conv_fwd_launch<16, 8, 4>(s, in, B, ci, cip, Wm, kp, co, cop, bias, out, L);
    else if (L >= 8 && conv_fwd_lds_t<8, 8, 4>(cip, cop) <= lim && conv_blocks(B, L, 8, 8, 4) >= kMinConvBlocks)
        conv_fwd_launch<8, 8, 4>(s, in, B, ci, cip, Wm, kp, co, cop, bias, out, L);
    else if (conv_fwd_lds_t<8, 4, 4>(cip, cop) <= lim && conv_blocks(B, L, 8, 4, 4) >= kMinConvBlocks)
        conv_fwd_launch<8, 4, 4>(s, in, B, ci, cip, Wm, kp, co, cop, bias, out, L);
    else
        conv_fwd_launch<8, 4, 2>(s, in, B, ci, cip, Wm, kp, co, cop, bias, out, L);
}

// Width of the weight gradient's site tiles in units of 8: the widest of 32, 16 and 8 sites that
// pads the box by at most an eighth (a wide tile stages fewer neighbours of its rows and gives
// each wave more K chunks per barrier); 8 where rows are not read four sites at a time.
static int wgrad_xc(int L)
{
    if (L % 4) return 1;
    for (int xc = 4; xc > 1; xc /= 2)
        if (((L + 8 * xc - 1) / (8 * xc) * 8 * xc - L) * 8 <= L) return xc;
    return 1;
}

static int wgrad_tiles(int B, int L)
{
    const int xw = 8 * wgrad_xc(L);
    return B * ((L + xw - 1) / xw) * ((L + kWgTY - 1) / kWgTY) * ((L + kWgTZ - 1) / kWgTZ);
}

// Slices of a layer's weight gradient: kWgBlocks blocks (channel octets x slices), each with at
// least one tile.  A level's layers share a launch, so one block per CU and layer fills the
// chip; more blocks write more partials (64^3, batch 2, five layers and the sums of all: 512
// blocks 90 + 22 us, 256 80 + 14).
constexpr int kWgBlocks = 256;
int net_wgrad_slices(int B, int L, int ci)
{
    return std::min(wgrad_tiles(B, L), std::max(1, kWgBlocks / ((ci + 7) / 8)));
}
long long net_wgrad_part(int slices, int ci, int co) { return (long long)((ci + 7) / 8) * slices * co * kWgElems; }

void net_conv_wgrad(hipStream_t s, WgradJobs &W, int B, int L)
{
    int blocks = 0, co = 0;
    for (int k = 0; k < W.n; ++k) {
        W.j[k].block0 = blocks;
        blocks += (W.j[k].ci + 7) / 8 * W.j[k].slices;
        co = std::max(co, W.j[k].co);
    }
    // above 16 outputs the accumulators leave no registers for the widest tile's staging
    const int xc = co > 16 ? std::min(wgrad_xc(L), 2) : wgrad_xc(L), xw = 8 * xc;
    const int tx = (L + xw - 1) / xw, ty = (L + kWgTY - 1) / kWgTY, tz = (L + kWgTZ - 1) / kWgTZ;
    auto go = [&](auto VEC, auto XC, auto MT) {
        hipLaunchKernelGGL((k_conv_wgrad<VEC(), XC(), MT()>), dim3(blocks), dim3(256), 0, s, W, L, tx, ty, tx * ty * tz,
                           B * tx * ty * tz);
    };
    auto width = [&](auto MT) {
        if (L % 4) go(std::false_type(), std::integral_constant<int, 1>(), MT);
        else if (xc == 2) go(std::true_type(), std::integral_constant<int, 2>(), MT);
        else go(std::true_type(), std::integral_constant<int, 1>(), MT);
    };
    if (xc == 4) go(std::true_type(), std::integral_constant<int, 4>(), std::integral_constant<int, 1>());
    else if (co <= 16) width(std::integral_constant<int, 1>());
    else width(std::integral_constant<int, 2>());
}

void net_wgrad_sum(hipStream_t s, WgradSums &W, const float *part, const double *bpart, float *grad)
{
    int blocks = 0;
    for (int l = 0; l < W.n; ++l) {
        W.l[l].block0 = blocks;
        blocks += (int)nb((long long)((W.l[l].ci + 7) / 8) * W.l[l].co * kWgElems, 32) + 1;
    }
    hipLaunchKernelGGL(k_wgrad_sum, dim3(blocks), dim3(256), 0, s, W, part, bpart, grad);
}

void net_pool_bwd(hipStream_t s, const float *dout, const ConvGive &to, int L, long long n_in)
{
    hipLaunchKernelGGL(k_pool_bwd, dim3(nb(n_in / 2, 256)), dim3(256), 0, s, dout, to, L, n_in);
}

void net_up_bwd(hipStream_t s, const float *dout, const ConvGive &to, int L, long long n_in)
{
    hipLaunchKernelGGL(k_up_bwd, dim3(nb(n_in, 256)), dim3(256), 0, s, dout, to, L, n_in);
}

int net_mse(hipStream_t s, const float *p, const float *t, float *dp, long long n, float inv_count, double *part)
{
    const int blocks = (int)nb(n, 256);
    hipLaunchKernelGGL(k_mse, dim3(blocks), dim3(256), 0, s, p, t, dp, n, inv_count, part);
    return blocks;
}

void net_adam(hipStream_t s, float *w, const float *g, float *m, float *v, long long n, float lr, float b1, float b2,
              float eps, float c1, float c2)
{
    hipLaunchKernelGGL(k_adam, dim3(nb(n, 256)), dim3(256), 0, s, w, g, m, v, n, lr, b1, b2, eps, c1, c2);
}

void net_stage_weights(hipStream_t s, const float *W, int co, int ci, int cip, int kp, int cop_rows, __bf16 *Wm,
                       int cip_t, int kp_t, int cop_rows_t, __bf16 *Wt)
{
    const long long n = (long long)cop_rows * kp + (long long)cop_rows_t * kp_t;
    hipLaunchKernelGGL(k_stage_weights, dim3(nb(n, 256)), dim3(256), 0, s, W, co, ci, cip, kp, cop_rows, Wm, cip_t,
                       kp_t, cop_rows_t, Wt);
}

void net_warm_input(hipStream_t s, const double *phi, const double *h0, const double *h1, int nsp, long long V,
                    int mode, double *part, int max_parts, double *rms, float *x)
{
    const long long n = (long long)nsp * V;
    if (mode != 0) {
        const int nparts = (int)std::min<long long>(max_parts, std::max<long long>(1, nb(n, 256)));
        hipLaunchKernelGGL(k_delta_sumsq, dim3(nparts), dim3(256), 0, s, phi, h0, h1, n, mode, part);
        hipLaunchKernelGGL(k_delta_rms, dim3(1), dim3(256), 0, s, part, nparts, n, rms);
    }
    hipLaunchKernelGGL(k_net_input, dim3(nb(n, 256)), dim3(256), 0, s, phi, h0, h1, n, mode, rms, x);
}

void net_warm_apply(hipStream_t s, double *w, const float *p, long long V, int mode, const double *rms,
                    const double *wh0, const double *wh1)
{
    hipLaunchKernelGGL(k_warm_apply, dim3(nb(2 * V, 256)), dim3(256), 0, s, w, p, 2 * V, mode, rms, wh0, wh1);
}

void net_shift_fields(hipStream_t s, double *w, const double *wh0, const double *wh1, long long n)
{
    hipLaunchKernelGGL(k_shift_fields, dim3(nb(n, 256)), dim3(256), 0, s, w, wh0, wh1, n);
}

void net_sample(hipStream_t s, const double *phi, const double *phi0, const double *phi1, const double *w,
                const double *w0, const double *w1, int nsp, long long V, int mode, double *part, int max_parts,
                double *rms, float *x, float *y)
{
    net_warm_input(s, phi, phi0, phi1, nsp, V, mode, part, max_parts, rms, x);
    hipLaunchKernelGGL(k_net_target, dim3(nb(2 * V, 256)), dim3(256), 0, s, w, w0, w1, 2 * V, mode, rms, y);
}

void net_channel_moments(hipStream_t s, const float *x, int batch, int C, long long V, double *part, int nblk,
                         double *out)
{
    hipLaunchKernelGGL(k_channel_sums, dim3(C, nblk), dim3(256), 0, s, x, batch, C, V, nblk, part);
    hipLaunchKernelGGL(k_channel_finish, dim3(1), dim3(64), 0, s, part, C, nblk, (double)batch * (double)V, out);
}

void net_affine(hipStream_t s, float *x, int C, long long V, long long n, const float *shift, const float *scale)
{
    hipLaunchKernelGGL(k_affine, dim3(nb(n, 256)), dim3(256), 0, s, x, C, V, n, shift, scale);
}


}  // namespace hsf
