// rg_corr.hpp -- coarse-fine flux correction of one coarse cell.
//
// Paper Sec. 3 (conservative update across refinement boundaries).  A coarse
// cell receives the fluxes owed by the fine octs on its six sides in the
// order of the octs' sides x-, x+, y-, y+, z-, z+.  Six passes, one per side,
// need no atomics but cost six launches of about 5 us and read every list
// row six times; here one thread owns the cell: the one of the first side
// that contributes, which then adds all sides in that order (the same bits)
// and, in a chained step, takes the cell's CFL limit of the next step.
//
// A fine oct o across whose side s the coarse cell C lies is at C - dir(s),
// in octs; the oct owing across side t is at o + dir(s) - dir(t), an entry of
// o's own list unless t is the side opposite to s.  That oct, two steps away,
// exists only where the cell beyond C is split too (its son bit tells), and
// is then looked up in the sorted keys; rare: a strip of unrefined cells one
// cell wide.
#pragma once

#include "rg_internal.hpp"
#include "rg_math.hpp"

namespace rg {
namespace {

struct CorrTree {
    double *unew;
    const double *corr;
    int64_t corr_base;
    const int32_t *nbr27;
    const uint32_t *son;
    const uint64_t *keys;
    int64_t begin[RG_MAX_LEVEL + 2];
    int lmin, lmax;
    double gamma, cfl;
};

__device__ __forceinline__ int corr_step(int side)
{
    const int step = side < 2 ? 1 : (side < 4 ? 3 : 9);
    return (side & 1) ? step : -step;
}

// the oct of level l two octs beyond oct o across `side`, -1 if there is none
template <typename T> __device__ inline int64_t corr_opposite(const T &a, int64_t o, int64_t C, int side, int l)
{
    const int ax = side >> 1, hi = side & 1;
    // the cell beyond C and whether it has a child oct
    int64_t P = C >> 3;
    const int q = static_cast<int>(C & 7);
    if (((q >> ax) & 1) == hi) P = a.nbr27[27 * P + 13 + corr_step(side)];
    if (P < 0 || !((a.son[P] >> (q ^ (1 << ax))) & 1u)) return -1;
    int32_t p[3], lev;
    key_coords(a.keys[o], p[0], p[1], p[2], lev);
    const int32_t n = int32_t(1) << (l - 1);
    p[ax] = (p[ax] + (hi ? 2 : -2) + 2 * n) & (n - 1);
    const uint64_t want = oct_key(p[0], p[1], p[2], l);
    int64_t lo = a.begin[l], up = a.begin[l + 1];
    while (lo < up) {
        const int64_t m = lo + (up - lo) / 2;
        if (a.keys[m] < want) lo = m + 1;
        else up = m;
    }
    return lo < a.begin[l + 1] && a.keys[lo] == want ? lo : -1;
}

// Corrects the coarse cell across `side` of oct o if this is its first side;
// with dt, also lowers best to the cell's CFL limit (and tracks non-finite
// values in nf, see track_finite).
template <typename T>
__device__ inline void correct_cell(const T &a, int64_t o, int side, bool dt, double &best, double &nf)
{
    const int32_t *nb = a.nbr27 + 27 * o;
    const int32_t e = nb[13 + corr_step(side)];
    if (!(e < 0 && e != RG_NBR_OUTSIDE)) return;
    const int64_t C = -1 - int64_t(e);
    int64_t from[6];
    bool first = true;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        from[t] = t == side ? o : ((t >> 1) == (side >> 1) ? -1 : nb[13 + corr_step(side) - corr_step(t)]);
        if (t < side && from[t] >= 0) first = false;
    }
    if (!first) return;
    int l = a.lmin;
    while (l < a.lmax && o >= a.begin[l + 1]) ++l;
    const int64_t opp = corr_opposite(a, o, C, side, l);
    if (opp >= 0 && (side & 1)) return;
    double U[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) U[v] = a.unew[NV * C + v];
#pragma unroll
    for (int t = 0; t < 6; ++t) {
        const int64_t f = t == (side ^ 1) ? opp : from[t];
        if (f < 0) continue;
        const double *c = a.corr + 30 * (f - a.corr_base) + NV * t;
#pragma unroll
        for (int v = 0; v < NV; ++v) U[v] = U[v] + c[v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) a.unew[NV * C + v] = U[v];
    if (dt) {
        const double dx = ldexp(1.0, -(l - 1));
        double W[NV];
        prim64(U, a.gamma, W);
        const double cs = sqrt_pos(div_pos(a.gamma * W[4], W[0]));
        const double sp = ((fabs(W[1]) + fabs(W[2])) + fabs(W[3])) + 3.0 * cs;
        const double cd = a.cfl * (dx / sp);
        if (cd < best) best = cd;
        track_finite(nf, sp, U);
    }
}

// minimum over the workgroup of `threads` threads, folded into *dt
__device__ __forceinline__ void fold_block(double best, double nf, double *s_min, int threads, unsigned long long *dt,
                                           HashHeader *hdr)
{
    best = nonfinite_limit(best, nf);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const double o = __shfl_xor(best, off, 64);
        best = o < best ? o : best;
    }
    if ((threadIdx.x & 63) == 0) s_min[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = s_min[0];
        for (int k = 1; k < threads / 64; ++k) m = s_min[k] < m ? s_min[k] : m;
        fold_min(dt, m, hdr);
    }
}

}  // namespace
}  // namespace rg
