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
// trips.  kTailOcts: two doubles per cell and 14 bytes per oct in the 160 KB
// of LDS of a compute unit: the complete levels 1..4 (585 octs; one more
// would be 4096) and levels of up to about a thousand octs of a graded tree,
// whose 12 passes per cycle then cost no launches.
#pragma once

#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kTailOcts = 1120;
constexpr int kTailThreads = 1024;
constexpr int kTailPlane = kTailOcts + 16;   // octs of a cell plane: 16 modulo 32, see TailSmem

struct TailArgs {
    double *e;                // per cell: corrections (the potential on a unigrid's finest level)
    const double *f;          // right-hand sides of level m0
    const double *diag;       // Gauss-Seidel diagonals, 0 on cells outside; null: 6 everywhere
    const int32_t *nbr;       // [..][27] same-level octs, -1 if absent
    const int32_t *father;    // father cell of each oct
    int64_t begin[RG_MAX_LEVEL + 2];   // octs of level m: [begin[m], begin[m + 1])
    int m0, lcoarse, nu1, nu2, ncoarse;
};

// Values by cell of the oct, then by oct: lanes hold consecutive octs, so they
// touch consecutive words (eight values of an oct side by side would put the
// lanes of a wave 64 bytes apart, in 4 of the banks' 32 places).  The two
// cells of an odd and an even lane are an odd number of planes apart, and a
// plane is half the banks' width longer than a multiple of it.
struct TailSmem {
    double e[8 * kTailPlane];        // the oct after the last stands for absent neighbours: zeros
    double f[8 * kTailPlane];
    uint16_t nb[6][kTailOcts];       // face neighbours x-, x+, y-, y+, z-, z+
    uint16_t father[kTailOcts];      // father cell (8 oct + c)
};
static_assert(kTailPlane % 32 == 16 && sizeof(TailSmem) <= 160 * 1024, "tail layout");

__device__ __forceinline__ int tail_at(int o, int c) { return c * kTailPlane + o; }

// cell k (0..3) of colour 0 (even coordinate sum: 0, 3, 5, 6) or 1 (1, 2, 4, 7)
__device__ __forceinline__ int colour_cell(int colour, int k) { return ((k << 1) | ((k ^ (k >> 1)) & 1)) ^ colour; }

// sum of the six face neighbours of cell c of local oct o, in the order x-,
// x+, y-, y+, z-, z+ (cells outside and absent ones hold 0)
__device__ __forceinline__ double tail_sum6(const TailSmem &S, int o, int c)
{
    double v[6];
#pragma unroll
    for (int side = 0; side < 6; ++side) {
        const int ax = side >> 1, hi = side & 1;
        v[side] = S.e[tail_at(((c >> ax) & 1) == hi ? int(S.nb[side][o]) : o, c ^ (1 << ax))];
    }
    return ((((v[0] + v[1]) + v[2]) + v[3]) + v[4]) + v[5];
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
    if (__builtin_expect(!(ax > 1e-250 && ax < 1e250), 0)) {
        if (x == 0.0) return x;   // common where the right-hand side is zero; d > 0
        return x / d;
    }
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-d, q, x), y, q);
    return __builtin_fma(__builtin_fma(-d, q, x), y, q);
}

// a cell held by a thread for all passes over a level: where it and its six
// neighbours are in S.e, h^2 f, the diagonal and its reciprocal
template <bool DIAG> struct TailCell {
    int at, nb[6];
    double hf, d, y;

    // diag: of the tail's first oct
    __device__ __forceinline__ void set(const TailSmem &S, const double *__restrict__ diag, int o, int c, double h2)
    {
        at = tail_at(o, c);
#pragma unroll
        for (int side = 0; side < 6; ++side) {
            const int ax = side >> 1, hi = side & 1;
            nb[side] = tail_at(((c >> ax) & 1) == hi ? int(S.nb[side][o]) : o, c ^ (1 << ax));
        }
        hf = h2 * S.f[at];
        d = DIAG ? diag[8 * o + c] : 6.0;
        y = 1.0 / d;
    }

    __device__ __forceinline__ void relax(TailSmem &S) const
    {
        double v[6];
#pragma unroll
        for (int side = 0; side < 6; ++side) v[side] = S.e[nb[side]];
        const double x = (((((v[0] + v[1]) + v[2]) + v[3]) + v[4]) + v[5]) - hf;
        if (!DIAG || d != 0.0) S.e[at] = div_by(x, d, y);
    }
};

template <int CTRL> __device__ __forceinline__ double dpp(double x)
{
    return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                            __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
}

// Sweeps over an oct that is its own neighbour on every side (level 1 of a
// periodic box, the coarsest level of 50 sweeps by default): lane c of eight
// holds cell c, whose neighbours along axis a are both cell c ^ (1 << a), so a
// pass is lane swaps and arithmetic, without LDS (about a third of the latency
// of a pass through it; 13 of the 40 us the levels 1-4 took).
template <bool DIAG>
__device__ __forceinline__ void tail_sweeps_one(TailSmem &S, const double *__restrict__ diag, int o, double h2,
                                                int sweeps)
{
    const int c = threadIdx.x;
    if (c < 8) {
        const int at = tail_at(o, c);
        const bool red = ((c ^ (c >> 1) ^ (c >> 2)) & 1) == 0;
        const double hf = h2 * S.f[at], d = DIAG ? diag[8 * o + c] : 6.0, y = 1.0 / d;
        const bool inside = !DIAG || d != 0.0;
        double e = S.e[at];
        if (__ballot(inside) == 0) sweeps = 0;   // a small refined region: no cell of this level is inside
        for (int p = 0; p < 2 * sweeps; ++p) {
            const double vx = dpp<0xB1>(e), vy = dpp<0x4E>(e);   // quad permutations c ^ 1, c ^ 2
            const double vz = dpp<0x1B>(dpp<0x141>(e));          // reversed in eight, then in four: c ^ 4
            const double x = (((((vx + vx) + vy) + vy) + vz) + vz) - hf;
            const double q = div_by(x, d, y);
            e = inside && red == ((p & 1) == 0) ? q : e;
        }
        S.e[at] = e;
    }
    __syncthreads();
}

// sweeps over the local octs [ob, ob + n)
template <bool DIAG>
__device__ __forceinline__ void tail_sweeps(TailSmem &S, const double *__restrict__ diag, int ob, int n, double h2,
                                            int sweeps)
{
    const int t = threadIdx.x;
    if (n == 1 && S.nb[0][ob] == ob && S.nb[2][ob] == ob && S.nb[4][ob] == ob) {
        tail_sweeps_one<DIAG>(S, diag, ob, h2, sweeps);
        return;
    }
    if (4 * n <= 64) {
        // one wave holds a colour: no barrier between the passes, the LDS
        // operations of a wave are done in order
        if (t < 64) {
            TailCell<DIAG> red, black;
            const int o = ob + (t < 4 * n ? t >> 2 : 0);
            red.set(S, diag, o, colour_cell(0, t & 3), h2);
            black.set(S, diag, o, colour_cell(1, t & 3), h2);
            if (__ballot(red.d != 0.0 || black.d != 0.0) == 0) sweeps = 0;
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
    // half an oct per thread and round: two cells of either colour, kept in
    // registers where one round holds the level
    const bool one = 2 * n <= kTailThreads;
    TailCell<DIAG> red[2], black[2];
    auto set = [&](int i, bool r, bool b) {
        const int o = ob + (i >> 1), k = 2 * (i & 1);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (r) red[j].set(S, diag, o, colour_cell(0, k + j), h2);
            if (b) black[j].set(S, diag, o, colour_cell(1, k + j), h2);
        }
    };
    if (one) set(t < 2 * n ? t : 0, true, true);
    for (int sw = 0; sw < sweeps; ++sw) {
        for (int i = t; i < 2 * n; i += kTailThreads) {
            if (!one) set(i, true, false);
            red[0].relax(S);
            red[1].relax(S);
        }
        __syncthreads();
        for (int i = t; i < 2 * n; i += kTailThreads) {
            if (!one) set(i, false, true);
            black[0].relax(S);
            black[1].relax(S);
        }
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
    __shared__ TailSmem S;
    const int tid = threadIdx.x;
    const int64_t base = A.begin[A.lcoarse];
    const int n_oct = static_cast<int>(A.begin[A.m0 + 1] - base);
    const int top = static_cast<int>(A.begin[A.m0] - base);   // first oct of level m0
    for (int i = tid; i < 8 * n_oct; i += kTailThreads) {
        const bool own = i >= 8 * top;
        S.e[tail_at(i >> 3, i & 7)] = own ? A.e[8 * base + i] : 0.0;
        S.f[tail_at(i >> 3, i & 7)] = own ? A.f[8 * base + i] : 0.0;
    }
    if (tid < 8) S.e[tail_at(n_oct, tid)] = 0.0;
    const double *diag = DIAG ? A.diag + 8 * base : nullptr;
    for (int i = tid; i < 6 * n_oct; i += kTailThreads) {
        const int o = i / 6, side = i - 6 * o;
        const int step = side < 2 ? 1 : (side < 4 ? 3 : 9);
        const int32_t n = A.nbr[27 * (base + o) + 13 + ((side & 1) ? step : -step)];
        S.nb[side][o] = static_cast<uint16_t>(n >= 0 ? n - base : n_oct);
    }
    const int first_child = static_cast<int>(A.begin[A.lcoarse + 1] - base);   // no fathers on lcoarse
    for (int o = first_child + tid; o < n_oct; o += kTailThreads)
        S.father[o] = static_cast<uint16_t>(A.father[base + o] - 8 * base);
    __syncthreads();

    for (int m = A.m0; m > A.lcoarse; --m) {
        const int ob = static_cast<int>(A.begin[m] - base), n = static_cast<int>(A.begin[m + 1] - base) - ob;
        const double h2 = ldexp(1.0, -2 * m);
        tail_sweeps<DIAG>(S, diag, ob, n, h2, A.nu1);
        for (int t = tid; t < 8 * n; t += kTailThreads) {   // eight lanes an oct
            const int o = ob + (t >> 3), c = t & 7, cell = tail_at(o, c);
            const double d = DIAG ? diag[8 * o + c] : 6.0;
            const double lap = (tail_sum6(S, o, c) - d * S.e[cell]) / h2;
            double r = DIAG && d == 0.0 ? 0.0 : S.f[cell] - lap;
            r = r + __shfl_xor(r, 1, 64);
            r = r + __shfl_xor(r, 2, 64);
            r = r + __shfl_xor(r, 4, 64);
            if (c == 0) S.f[tail_at(S.father[o] >> 3, S.father[o] & 7)] = 0.125 * r;
        }
        __syncthreads();
    }
    {
        const int n = static_cast<int>(A.begin[A.lcoarse + 1] - base);
        tail_sweeps<DIAG>(S, diag, 0, n, ldexp(1.0, -2 * A.lcoarse), A.ncoarse);
    }
    for (int m = A.lcoarse + 1; m <= A.m0; ++m) {
        const int ob = static_cast<int>(A.begin[m] - base), n = static_cast<int>(A.begin[m + 1] - base) - ob;
        for (int t = tid; t < 8 * n; t += kTailThreads) {
            const int o = ob + (t >> 3), c = t & 7, cell = tail_at(o, c);
            if (DIAG && diag[8 * o + c] == 0.0) continue;
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
                v[b] = S.e[tail_at(nn >= 0 ? static_cast<int>(nn - base) : n_oct, q ^ b)];
            }
            const double w = ((((((27.0 * v[0] + 9.0 * v[1]) + 9.0 * v[2]) + 9.0 * v[4]) + 3.0 * v[3]) + 3.0 * v[5]) +
                              3.0 * v[6]) + v[7];
            S.e[cell] = S.e[cell] + 0.015625 * w;
        }
        __syncthreads();
        tail_sweeps<DIAG>(S, diag, ob, n, ldexp(1.0, -2 * m), A.nu2);
    }
    for (int i = 8 * top + tid; i < 8 * n_oct; i += kTailThreads) A.e[8 * base + i] = S.e[tail_at(i >> 3, i & 7)];
}

}  // namespace
}  // namespace rg
