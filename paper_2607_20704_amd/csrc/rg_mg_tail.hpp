// rg_mg_tail.hpp -- the small levels of a multigrid V-cycle in one workgroup.
//
// Paper Sec. 5 (V-cycles).  Shared by the unigrid solver and the solver level
// by level.  The coarse levels that hold at most kTailOcts octs in all run
// their whole part of a V-cycle in one workgroup with everything in LDS:
// corrections, right-hand sides, diagonals and face-neighbour indices.
//
// What bounds it: a chain of dependent passes (two per sweep, about 30 on
// the levels 2..4 and 100 on a coarsest level of 50 sweeps), each as long as
// its latency.  One kernel per pass costs about 5 us; passes through global
// memory in one workgroup cost 1-2 us each (150 us per cycle for the levels
// 1..4 of a unigrid); from LDS a pass costs its barrier and a few LDS round
// trips.  kTailOcts: three doubles per cell and 14 bytes per oct in the
// 160 KB of LDS of a compute unit, and enough for the complete levels 1..4
// (585 octs); one more complete level would be 4096 octs.
#pragma once

#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kTailOcts = 640;
constexpr int kTailThreads = 1024;

struct TailArgs {
    double *e;                // per cell: corrections (the potential on a unigrid's finest level)
    const double *f;          // right-hand sides of level m0
    const double *diag;       // Gauss-Seidel diagonals, 0 on cells outside; null: 6 everywhere
    const int32_t *nbr;       // [..][27] same-level octs, -1 if absent
    const int32_t *father;    // father cell of each oct
    int64_t begin[RG_MAX_LEVEL + 2];   // octs of level m: [begin[m], begin[m + 1])
    int m0, lcoarse, nu1, nu2, ncoarse;
};

template <bool DIAG> struct TailSmem {
    double e[8 * (kTailOcts + 1)];   // the last oct stands for absent neighbours: zeros
    double f[8 * kTailOcts];
    double diag[DIAG ? 8 * kTailOcts : 1];
    uint16_t nb[kTailOcts][6];       // face neighbours x-, x+, y-, y+, z-, z+
    uint16_t father[kTailOcts];      // father cell
};

// cell k (0..3) of colour 0 (even coordinate sum: 0, 3, 5, 6) or 1 (1, 2, 4, 7)
__device__ __forceinline__ int colour_cell(int colour, int k) { return ((k << 1) | ((k ^ (k >> 1)) & 1)) ^ colour; }

// sum of the six face neighbours of cell c of local oct o, in the order x-,
// x+, y-, y+, z-, z+ (cells outside and absent ones hold 0)
template <typename SM> __device__ __forceinline__ double tail_sum6(const SM &S, int o, int c)
{
    double v[6];
#pragma unroll
    for (int side = 0; side < 6; ++side) {
        const int ax = side >> 1, hi = side & 1;
        const int n = ((c >> ax) & 1) == hi ? S.nb[o][side] : o;
        v[side] = S.e[8 * n + (c ^ (1 << ax))];
    }
    return ((((v[0] + v[1]) + v[2]) + v[3]) + v[4]) + v[5];
}

template <bool DIAG, typename SM>
__device__ __forceinline__ void tail_relax(SM &S, int o, int c, double h2)
{
    const int cell = 8 * o + c;
    const double d = DIAG ? S.diag[cell] : 6.0;
    if (DIAG && d == 0.0) return;
    S.e[cell] = (tail_sum6(S, o, c) - h2 * S.f[cell]) / d;
}

// x / d, correctly rounded, with y = 1 / d rounded to nearest: q = x y is at
// most two units off, the first correction makes it faithful, and the second,
// q + (x - d q) y, rounds correctly (P. Markstein, IBM J. Res. Dev. 34, 1990)
// as long as the remainder is exact, which it is away from the ends of the
// exponent range; those (and infinities and NaN) take the division itself.
// 5 dependent instructions instead of a division's scaled sequence.
__device__ __forceinline__ double div_by(double x, double d, double y)
{
    const double ax = fabs(x);
    if (__builtin_expect(!(ax > 1e-250 && ax < 1e250), 0)) return x / d;
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-d, q, x), y, q);
    return __builtin_fma(__builtin_fma(-d, q, x), y, q);
}

// a cell held by a thread for all passes over a level: where it and its six
// neighbours are in S.e, h^2 f, the diagonal and its reciprocal
template <bool DIAG> struct TailCell {
    int at, nb[6];
    double hf, d, y;

    template <typename SM> __device__ __forceinline__ void set(const SM &S, int o, int c, double h2)
    {
        at = 8 * o + c;
#pragma unroll
        for (int side = 0; side < 6; ++side) {
            const int ax = side >> 1, hi = side & 1;
            nb[side] = 8 * (((c >> ax) & 1) == hi ? int(S.nb[o][side]) : o) + (c ^ (1 << ax));
        }
        hf = h2 * S.f[at];
        d = DIAG ? S.diag[at] : 6.0;
        y = 1.0 / d;
    }

    template <typename SM> __device__ __forceinline__ void relax(SM &S) const
    {
        double v[6];
#pragma unroll
        for (int side = 0; side < 6; ++side) v[side] = S.e[nb[side]];
        const double x = (((((v[0] + v[1]) + v[2]) + v[3]) + v[4]) + v[5]) - hf;
        if (!DIAG || d != 0.0) S.e[at] = div_by(x, d, y);
    }
};

// sweeps over the local octs [ob, ob + n)
template <bool DIAG, typename SM>
__device__ __forceinline__ void tail_sweeps(SM &S, int ob, int n, double h2, int sweeps)
{
    const int t = threadIdx.x;
    if (4 * n <= 64) {
        // one wave holds a colour: no barrier between the passes, the LDS
        // operations of a wave are done in order
        if (t < 64) {
            TailCell<DIAG> red, black;
            const int o = ob + (t < 4 * n ? t >> 2 : 0);
            red.set(S, o, colour_cell(0, t & 3), h2);
            black.set(S, o, colour_cell(1, t & 3), h2);
            for (int sw = 0; sw < sweeps; ++sw) {
                if (t < 4 * n) red.relax(S);
                __threadfence_block();
                __builtin_amdgcn_wave_barrier();
                if (t < 4 * n) black.relax(S);
                __threadfence_block();
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        return;
    }
    if (2 * n <= kTailThreads) {
        // half an oct per thread: two cells of either colour
        const bool on = t < 2 * n;
        const int o = ob + (on ? t >> 1 : 0), k = 2 * (t & 1);
        TailCell<DIAG> red[2], black[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            red[i].set(S, o, colour_cell(0, k + i), h2);
            black[i].set(S, o, colour_cell(1, k + i), h2);
        }
        for (int sw = 0; sw < sweeps; ++sw) {
            if (on) {
                red[0].relax(S);
                red[1].relax(S);
            }
            __syncthreads();
            if (on) {
                black[0].relax(S);
                black[1].relax(S);
            }
            __syncthreads();
        }
        return;
    }
    for (int p = 0; p < 2 * sweeps; ++p) {
        for (int i = t; i < 4 * n; i += kTailThreads)
            tail_relax<DIAG>(S, ob + (i >> 2), colour_cell(p & 1, i & 3), h2);
        __syncthreads();
    }
}

// Level m0's part of a V-cycle and everything below it: nu1 sweeps, residual
// restricted as the mean of 8 children (summed pairwise), the level below
// from zero (ncoarse sweeps on lcoarse), trilinear interpolation added, nu2
// sweeps; the passes and the order of every sum are those of the per-level
// kernels, so the bits are the same.
template <bool DIAG> __global__ __launch_bounds__(kTailThreads) void k_mg_tail(TailArgs A)
{
    __shared__ TailSmem<DIAG> S;
    const int tid = threadIdx.x;
    const int64_t base = A.begin[A.lcoarse];
    const int n_oct = static_cast<int>(A.begin[A.m0 + 1] - base);
    const int top = static_cast<int>(A.begin[A.m0] - base);   // first oct of level m0
    for (int i = tid; i < 8 * n_oct; i += kTailThreads) {
        const bool own = i >= 8 * top;
        S.e[i] = own ? A.e[8 * base + i] : 0.0;
        S.f[i] = own ? A.f[8 * base + i] : 0.0;
        if constexpr (DIAG) S.diag[i] = A.diag[8 * base + i];
    }
    if (tid < 8) S.e[8 * n_oct + tid] = 0.0;
    for (int i = tid; i < 6 * n_oct; i += kTailThreads) {
        const int o = i / 6, side = i - 6 * o;
        const int step = side < 2 ? 1 : (side < 4 ? 3 : 9);
        const int32_t n = A.nbr[27 * (base + o) + 13 + ((side & 1) ? step : -step)];
        S.nb[o][side] = static_cast<uint16_t>(n >= 0 ? n - base : n_oct);
    }
    const int first_child = static_cast<int>(A.begin[A.lcoarse + 1] - base);   // no fathers on lcoarse
    for (int o = first_child + tid; o < n_oct; o += kTailThreads)
        S.father[o] = static_cast<uint16_t>(A.father[base + o] - 8 * base);
    __syncthreads();

    for (int m = A.m0; m > A.lcoarse; --m) {
        const int ob = static_cast<int>(A.begin[m] - base), n = static_cast<int>(A.begin[m + 1] - base) - ob;
        const double h2 = ldexp(1.0, -2 * m);
        tail_sweeps<DIAG>(S, ob, n, h2, A.nu1);
        for (int t = tid; t < 8 * n; t += kTailThreads) {   // eight lanes an oct
            const int o = ob + (t >> 3), c = t & 7, cell = 8 * o + c;
            const double d = DIAG ? S.diag[cell] : 6.0;
            const double lap = (tail_sum6(S, o, c) - d * S.e[cell]) / h2;
            double r = DIAG && d == 0.0 ? 0.0 : S.f[cell] - lap;
            r = r + __shfl_xor(r, 1, 64);
            r = r + __shfl_xor(r, 2, 64);
            r = r + __shfl_xor(r, 4, 64);
            if (c == 0) S.f[S.father[o]] = 0.125 * r;
        }
        __syncthreads();
    }
    {
        const int n = static_cast<int>(A.begin[A.lcoarse + 1] - base);
        tail_sweeps<DIAG>(S, 0, n, ldexp(1.0, -2 * A.lcoarse), A.ncoarse);
    }
    for (int m = A.lcoarse + 1; m <= A.m0; ++m) {
        const int ob = static_cast<int>(A.begin[m] - base), n = static_cast<int>(A.begin[m + 1] - base) - ob;
        for (int t = tid; t < 8 * n; t += kTailThreads) {
            const int o = ob + (t >> 3), c = t & 7, cell = 8 * o + c;
            if (DIAG && S.diag[cell] == 0.0) continue;
            const int C = S.father[o], P = C >> 3, q = C & 7;
            // the coarse cells C + {0, s}^3, s the side of C's centre that
            // c lies on; a step along axis a leaves the oct where s points
            // to the side that C is on
            int out[3];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int hi = (c >> a) & 1;
                const int step = a == 0 ? 1 : (a == 1 ? 3 : 9);
                out[a] = ((q >> a) & 1) == hi ? (hi ? step : -step) : 0;
            }
            double v[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int slot = 13 + ((b & 1) ? out[0] : 0) + ((b & 2) ? out[1] : 0) + ((b & 4) ? out[2] : 0);
                const int32_t nn = A.nbr[27 * (base + P) + slot];
                v[b] = S.e[8 * (nn >= 0 ? static_cast<int>(nn - base) : n_oct) + (q ^ b)];
            }
            const double w = ((((((27.0 * v[0] + 9.0 * v[1]) + 9.0 * v[2]) + 9.0 * v[4]) + 3.0 * v[3]) + 3.0 * v[5]) +
                              3.0 * v[6]) + v[7];
            S.e[cell] = S.e[cell] + 0.015625 * w;
        }
        __syncthreads();
        tail_sweeps<DIAG>(S, ob, n, ldexp(1.0, -2 * m), A.nu2);
    }
    for (int i = 8 * top + tid; i < 8 * n_oct; i += kTailThreads) A.e[8 * base + i] = S.e[i];
}

}  // namespace
}  // namespace rg
