// rg_mg_brick.hpp -- multigrid passes over a complete periodic level, one
// 8^3-oct brick (16^3 cells) per workgroup.
//
// Paper Sec. 5 (red-black Gauss-Seidel, residual restriction, trilinear
// prolongation).  A brick is a contiguous stretch of 512 octs of the Hilbert
// order; on a complete level the octs around it are found by evaluating the
// order, so no neighbour list is read.  A sweep reads the brick and a shell
// of one oct (two cells) into LDS, relaxes the red cells of the brick and of
// the face layer around it, then the brick's black cells, and writes the
// result to a second array (the shell of a neighbouring brick must still be
// the old state).  The red cells of the face layers are relaxed by both
// bricks that share them, from the same operands in the same order, so every
// bit is that of the two passes over the whole level.
//
// What bounds it: memory.  A colour pass of its own read each cell's list
// entries (13.5 bytes a cell), the potential and the right-hand side and
// wrote half of the potential: 75 bytes per cell and sweep (324 us on the
// 256^3 level).  Here a sweep moves 8 (10/8)^3 bytes of potential, 8 of
// right-hand side for the brick and 3 for the face layers, and 8 written: 35
// bytes, part of the shell from L2.  One sweep per pass over memory: two
// would need a shell of four cells, 24^3 cells for 16^3 (110 KB of LDS, one
// workgroup per compute unit) and as many bytes.
#pragma once

#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kMbT = 512;          // threads: one per oct of the brick
constexpr int kMbW = 20;           // tile side, cells
constexpr int kMbShell = 488;      // octs around the brick
enum { MB_SWEEP = 0, MB_PROLONG = 1, MB_RESTRICT = 2, MB_RESIDUAL = 3 };

struct MgBrickArgs {
    const double *src;     // potential of the level (first cell of the level)
    double *dst;           // MB_SWEEP, MB_PROLONG: the swept potential; MB_RESIDUAL: the residual
    const double *f;       // right-hand side of the level
    const double *ec;      // MB_PROLONG: correction of the level below, added first
    double *fc, *zc;       // MB_RESTRICT: right-hand side of the level below; its potential, set to zero
    int l;                 // level, >= 4
};

__device__ __forceinline__ int mb_pos(int x, int y, int z) { return (x + 2) + kMbW * ((y + 2) + kMbW * (z + 2)); }

// oct offset of cell c of an oct in the tile
__device__ __forceinline__ int mb_cell(int c) { return (c & 1) + kMbW * ((c >> 1) & 1) + kMbW * kMbW * (c >> 2); }

// trilinear interpolation of the coarse tile C (12^3 cells, offset 2) added to
// the 8 cells of the oct over coarse cell (x, y, z)
__device__ __forceinline__ void mb_prolong(const double *C, int x, int y, int z, double *v)
{
    const double *p = C + (x + 2) + 12 * ((y + 2) + 12 * (z + 2));
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const int s[3] = {(c & 1) ? 1 : -1, (c & 2) ? 12 : -12, (c & 4) ? 144 : -144};
        double e[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) e[b] = p[((b & 1) ? s[0] : 0) + ((b & 2) ? s[1] : 0) + ((b & 4) ? s[2] : 0)];
        const double w = ((((((27.0 * e[0] + 9.0 * e[1]) + 9.0 * e[2]) + 9.0 * e[4]) + 3.0 * e[3]) + 3.0 * e[5]) +
                          3.0 * e[6]) + e[7];
        v[c] = v[c] + 0.015625 * w;
    }
}

// sum of the six face neighbours (x-, x+, y-, y+, z-, z+) of cell c of the
// oct whose values are v and whose first cell is at p in the tile
__device__ __forceinline__ double mb_sum6(const double *T, int p, const double *v, int c)
{
    const int q = p + mb_cell(c);
    const double xm = (c & 1) ? v[c ^ 1] : T[q - 1], xp = (c & 1) ? T[q + 1] : v[c ^ 1];
    const double ym = (c & 2) ? v[c ^ 2] : T[q - kMbW], yp = (c & 2) ? T[q + kMbW] : v[c ^ 2];
    const double zm = (c & 4) ? v[c ^ 4] : T[q - kMbW * kMbW], zp = (c & 4) ? T[q + kMbW * kMbW] : v[c ^ 4];
    return ((((xm + xp) + ym) + yp) + zm) + zp;
}

template <int MODE> __global__ __launch_bounds__(kMbT, 4) void k_mg_brick(MgBrickArgs a)
{
    __shared__ double T[kMbW * kMbW * kMbW];
    __shared__ double C[MODE == MB_PROLONG ? 12 * 12 * 12 : 1];
    const int tid = threadIdx.x;
    const int nb = a.l - 1;
    const int64_t nbricks = int64_t(1) << (3 * (nb - 3));
    // consecutive bricks on one XCD, which share their shells in its L2
    const int64_t b = nbricks < 8 ? blockIdx.x : (blockIdx.x % 8) * (nbricks / 8) + blockIdx.x / 8;
    const int64_t o = 512 * b + tid;
    const uint32_t wrap = (uint32_t(1) << nb) - 1;
    uint32_t i, j, k;
    hilbert_point_bits(static_cast<uint64_t>(o), nb, i, j, k);
    const uint32_t bx = i & ~7u, by = j & ~7u, bz = k & ~7u;
    const int ox = i & 7, oy = j & 7, oz = k & 7;

    double v[8], f[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        v[c] = a.src[8 * o + c];
        f[c] = a.f[8 * o + c];
    }
    // one oct of the shell: two 10 x 10 plates, then rings of 36
    int sx, sy, sz;
    if (tid < 200) {
        sz = tid < 100 ? -1 : 8;
        const int r = tid < 100 ? tid : tid - 100;
        sx = r % 10 - 1;
        sy = r / 10 - 1;
    } else {
        const int t = tid - 200, r = t % 36;
        sz = t / 36;
        sy = r < 10 ? -1 : (r < 20 ? 8 : (r - 20) & 7);
        sx = r < 10 ? r - 1 : (r < 20 ? r - 11 : (r < 28 ? -1 : 8));
    }
    const int out = (sx < 0 || sx > 7) + (sy < 0 || sy > 7) + (sz < 0 || sz > 7);
    // corners are never read, edges not by a residual
    constexpr bool RES = MODE == MB_RESTRICT || MODE == MB_RESIDUAL;
    const bool shell = tid < kMbShell && out <= (RES ? 1 : 2);
    const bool face = tid < kMbShell && out == 1;
    const int ax = (sx < 0 || sx > 7) ? 0 : ((sy < 0 || sy > 7) ? 1 : 2);
    const int lo = ax == 0 ? sx < 0 : (ax == 1 ? sy < 0 : sz < 0);   // the layer next to the brick: bit ax of c = lo
    // the layer's two red cells
    const int r0 = lo ? (1 << ax) | (1 << ((ax + 1) % 3)) : 0;
    const int r1 = lo ? (1 << ax) | (1 << ((ax + 2) % 3)) : 7 ^ (1 << ax);
    double sf0 = 0.0, sf1 = 0.0;
    const int64_t so = static_cast<int64_t>(
        hilbert_index_bits((bx + sx) & wrap, (by + sy) & wrap, (bz + sz) & wrap, nb));
    if (!RES && face) {
        sf0 = a.f[8 * so + r0];
        sf1 = a.f[8 * so + r1];
    }
    const int p = mb_pos(2 * ox, 2 * oy, 2 * oz), sp = mb_pos(2 * sx, 2 * sy, 2 * sz);
    if constexpr (MODE == MB_PROLONG) {
        if (tid < 216) {
            const int cx = tid % 6 - 1, cy = (tid / 6) % 6 - 1, cz = tid / 36 - 1;
            const uint32_t cw = wrap >> 1;
            const int64_t co = static_cast<int64_t>(
                hilbert_index_bits(((bx >> 1) + cx) & cw, ((by >> 1) + cy) & cw, ((bz >> 1) + cz) & cw, nb - 1));
            const int p = (2 * cx + 2) + 12 * ((2 * cy + 2) + 12 * (2 * cz + 2));
#pragma unroll
            for (int c = 0; c < 8; ++c) C[p + (c & 1) + 12 * ((c >> 1) & 1) + 144 * (c >> 2)] = a.ec[8 * co + c];
        }
        __syncthreads();
    }
    if (shell) {
        double sv[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) sv[c] = a.src[8 * so + c];
        if constexpr (MODE == MB_PROLONG) mb_prolong(C, sx, sy, sz, sv);
#pragma unroll
        for (int c = 0; c < 8; ++c) T[sp + mb_cell(c)] = sv[c];
    }
    if constexpr (MODE == MB_PROLONG) mb_prolong(C, ox, oy, oz, v);
#pragma unroll
    for (int c = 0; c < 8; ++c) T[p + mb_cell(c)] = v[c];
    __syncthreads();
    const double h2 = ldexp(1.0, -2 * a.l);
    if constexpr (RES) {
        double r[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const double lap = (mb_sum6(T, p, v, c) - 6.0 * v[c]) / h2;
            r[c] = f[c] - lap;
        }
        if constexpr (MODE == MB_RESIDUAL) {
#pragma unroll
            for (int c = 0; c < 8; ++c) a.dst[8 * o + c] = r[c];
        } else {
            const int64_t fc = 8 * (o >> 3) + ((i & 1) + 2 * (j & 1) + 4 * (k & 1));
            a.fc[fc] = 0.125 * (((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7])));
            a.zc[fc] = 0.0;
        }
    } else {
        constexpr int red[4] = {0, 3, 5, 6}, black[4] = {1, 2, 4, 7};
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int c = red[n];
            v[c] = (mb_sum6(T, p, v, c) - h2 * f[c]) / 6.0;
            T[p + mb_cell(c)] = v[c];
        }
        if (face) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const int q = sp + mb_cell(n ? r1 : r0);
                const double s = ((((T[q - 1] + T[q + 1]) + T[q - kMbW]) + T[q + kMbW]) + T[q - kMbW * kMbW]) +
                                 T[q + kMbW * kMbW];
                T[q] = (s - h2 * (n ? sf1 : sf0)) / 6.0;
            }
        }
        __syncthreads();
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            const int c = black[n];
            v[c] = (mb_sum6(T, p, v, c) - h2 * f[c]) / 6.0;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) a.dst[8 * o + c] = v[c];
    }
}

template <int MODE> rg_status mg_brick(const MgBrickArgs &a, hipStream_t s)
{
    const unsigned bricks = static_cast<unsigned>(int64_t(1) << (3 * (a.l - 4)));
    k_mg_brick<MODE><<<bricks, kMbT, 0, s>>>(a);
    return launch_status("multigrid bricks");
}

// An even number of sweeps over complete level l (>= 4) from u back into u,
// through tmp; with ec, the correction of the level below is added first.
inline rg_status mg_brick_sweeps(double *u, double *tmp, const double *f, const double *ec, int l, int sweeps,
                                 hipStream_t s)
{
    MgBrickArgs a;
    a.f = f;
    a.ec = ec;
    a.fc = a.zc = nullptr;
    a.l = l;
    for (int k = 0; k < sweeps; ++k) {
        a.src = (k & 1) ? tmp : u;
        a.dst = (k & 1) ? u : tmp;
        RG_TRY(ec && k == 0 ? mg_brick<MB_PROLONG>(a, s) : mg_brick<MB_SWEEP>(a, s));
    }
    return RG_OK;
}

// residual of complete level l
inline rg_status mg_brick_residual(const double *u, const double *f, double *r, int l, hipStream_t s)
{
    MgBrickArgs a;
    a.src = u;
    a.dst = r;
    a.f = f;
    a.ec = nullptr;
    a.fc = a.zc = nullptr;
    a.l = l;
    return mg_brick<MB_RESIDUAL>(a, s);
}

// residual of complete level l restricted into the right-hand side of level
// l - 1, whose potential is set to zero
inline rg_status mg_brick_restrict(const double *u, const double *f, double *fc, double *zc, int l, hipStream_t s)
{
    MgBrickArgs a;
    a.src = u;
    a.dst = nullptr;
    a.f = f;
    a.ec = nullptr;
    a.fc = fc;
    a.zc = zc;
    a.l = l;
    return mg_brick<MB_RESTRICT>(a, s);
}

}  // namespace
}  // namespace rg
