// rg_oct.hpp -- per-oct hydro update body (one workgroup, G octs of one level).
//
// Paper Sec. 3: each oct is updated from a 6x6x6 stencil of uold (the oct
// and two ghost cells per side): primitive variables, reconstructed face
// states, HLLC fluxes, conservative update into unew.  Shared by the
// single-level kernel and the batched persistent kernel.
#pragma once

#include "rg_internal.hpp"
#include "rg_math.hpp"

namespace rg {
namespace {

// ---------------------------------------------------------------------------
// stencil tables (positions are cell offsets from the oct origin, -2..3)
// ---------------------------------------------------------------------------

constexpr int kOctW = 80;   // stencil cells: own 8, face layer 24, outer layer 24, edges 24
constexpr int kOctF = 36;   // faces: 3 axes x 3 planes x 4

__device__ __forceinline__ int nslot(int sx, int sy, int sz) { return (sx + 1) + 3 * (sy + 1) + 9 * (sz + 1); }

__device__ __forceinline__ int slot_of(int x) { return x < 0 ? -1 : (x > 1 ? 1 : 0); }

// face f = 12 a + 4 c + t1 + 2 t2 on axis a between cells c-1 and c along a;
// (t1, t2) are the other two axes in increasing order
__host__ __device__ constexpr int face_id(int a, int c, int t1, int t2) { return 12 * a + 4 * c + t1 + 2 * t2; }

// one word per item
struct StencilTables {
    // stencil cell: list entry (5 bits), cell within that oct (3), position +
    // 2 (3 bits per axis)
    uint32_t wcode[kOctW];
    // reconstructed cell (own 8, face layer 24): its neighbours' indices x-,
    // x+, y-, y+, z-, z+ (7 bits each)
    uint64_t rcode[32];
    // face-layer cell: the face it has a state for (6 bits), which side of it
    // the state is (0 left, 1 right), axis (2 bits)
    uint16_t fcode[24];
};

constexpr int tile_index(int x, int y, int z) { return (x + 2) + 6 * (y + 2) + 36 * (z + 2); }

constexpr StencilTables make_tables()
{
    StencilTables t{};
    int pos[kOctW][3] = {};
    int8_t index[216] = {};
    int n = 0;
    for (; n < 8; ++n)
        for (int a = 0; a < 3; ++a) pos[n][a] = (n >> a) & 1;
    // face layer (reconstructed) then outer layer, along each axis
    for (int layer = 0; layer < 2; ++layer)
        for (int a = 0; a < 3; ++a)
            for (int side = 0; side < 2; ++side)
                for (int q = 0; q < 4; ++q, ++n) {
                    const int t1 = a == 0 ? 1 : 0, t2 = a == 2 ? 1 : 2;
                    pos[n][a] = layer == 0 ? (side ? 2 : -1) : (side ? 3 : -2);
                    pos[n][t1] = q & 1;
                    pos[n][t2] = q >> 1;
                    // the high-side state of a cell below is left of face 0,
                    // the low-side state of a cell above right of face 2
                    if (layer == 0)
                        t.fcode[n - 8] = static_cast<uint16_t>(face_id(a, side ? 2 : 0, q & 1, q >> 1) | side << 6 |
                                                               a << 7);
                }
    // edge cells: two coordinates in {-1, 2}, the third in {0, 1}
    for (int a = 0; a < 3; ++a)        // the axis that stays inside
        for (int q = 0; q < 8; ++q, ++n) {
            const int u = a == 0 ? 1 : 0, v = a == 2 ? 1 : 2;
            pos[n][a] = q & 1;
            pos[n][u] = (q >> 1) & 1 ? 2 : -1;
            pos[n][v] = (q >> 2) & 1 ? 2 : -1;
        }
    for (int i = 0; i < kOctW; ++i) {
        index[tile_index(pos[i][0], pos[i][1], pos[i][2])] = static_cast<int8_t>(i);
        int slot = 13, cell = 0, where = 0;
        for (int a = 0, step = 1; a < 3; ++a, step *= 3) {
            const int c = pos[i][a];
            slot += c < 0 ? -step : (c > 1 ? step : 0);
            cell |= (c & 1) << a;
            where |= (c + 2) << (3 * a);
        }
        t.wcode[i] = static_cast<uint32_t>(slot | cell << 5 | where << 8);
    }
    for (int i = 0; i < 32; ++i) {
        const int x = pos[i][0], y = pos[i][1], z = pos[i][2];
        const int nb[6] = {index[tile_index(x - 1, y, z)], index[tile_index(x + 1, y, z)],
                           index[tile_index(x, y - 1, z)], index[tile_index(x, y + 1, z)],
                           index[tile_index(x, y, z - 1)], index[tile_index(x, y, z + 1)]};
        for (int k = 0; k < 6; ++k) t.rcode[i] |= static_cast<uint64_t>(nb[k]) << (7 * k);
    }
    return t;
}

__constant__ StencilTables c_tab = make_tables();

// ---------------------------------------------------------------------------
// the level kernel
// ---------------------------------------------------------------------------

// Variable v at the fine position of sub-cell `sub` of coarse cell C: C's
// value plus a quarter of each minmod slope, toward the position, taken from
// C's face neighbours (in C's oct, in the neighbouring oct, the coarser cell
// covering it, or C itself outside the domain).  Along each axis one neighbour
// lies in C's oct and the other across it; the three list entries, then the
// seven cells, are loaded together, two memory round trips in all.
__device__ __forceinline__ double coarse_ghost(const LevelArgs &a, int64_t C, int sub, int v)
{
    const int64_t P = C >> 3;
    const int q = static_cast<int>(C & 7);
    int32_t e[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int step = ax == 0 ? 1 : (ax == 1 ? 3 : 9);
        e[ax] = a.nbr27[27 * P + 13 + (((q >> ax) & 1) ? step : -step)];
    }
    const double uc = a.ucoarse[NV * C + v];
    double in[3], over[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) in[ax] = a.ucoarse[NV * (8 * P + (q ^ (1 << ax))) + v];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const double *src = e[ax] < 0 && e[ax] != RG_NBR_OUTSIDE ? a.ucoarse2 : a.ucoarse;
        const int64_t cell = e[ax] == RG_NBR_OUTSIDE ? C
                                                     : (e[ax] >= 0 ? 8 * int64_t(e[ax]) + (q ^ (1 << ax))
                                                                   : -1 - int64_t(e[ax]));
        over[ax] = src[NV * cell + v];
    }
    double u = uc;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const bool up = (q >> ax) & 1;   // C on its oct's high side: the neighbour across is the high one
        const double qq = ((sub >> ax) & 1) ? 0.25 : -0.25;
        const double lo = up ? in[ax] : over[ax], hi = up ? over[ax] : in[ax];
        u = u + qq * minmod<double>(uc - lo, hi - uc);
    }
    return u;
}

// Interpolated ghost cells of a workgroup's stencil: noted while the other
// cells are gathered, then formed one variable per thread, then turned into
// primitive variables.  Formed where the gather met them, five variables at
// once, they took 88 registers and every wave with one such lane through the
// whole interpolation (a subcycled step of the clumps of levels 6-9, mixed:
// 1566 us; like this 1388).
template <int N> struct GhostCells {
    double u[NV][N];            // their values
    int32_t n;
    int16_t cell[N];            // stencil index, sub-cell of the coarse cell above its 10 bits
    int32_t coarse[N];          // list entry of the coarse cell

    __device__ __forceinline__ void note(int it, int sub, int32_t e)
    {
        const uint64_t m = __ballot(1);
        const int rank = __popcll(m & ((uint64_t(1) << (threadIdx.x & 63)) - 1));
        int base = 0;
        if (rank == 0) base = atomicAdd(&n, __popcll(m));
        base = __builtin_amdgcn_readfirstlane(base);
        if (base + rank < N) {   // own cells are never ghosts
            cell[base + rank] = static_cast<int16_t>(it | sub << 10);
            coarse[base + rank] = e;
        }
    }
};

template <> struct GhostCells<0> {};

constexpr int kOctGhosts = kOctW - 8;   // stencil cells that may be ghosts

template <typename R, int G, bool GH = false> struct Smem {
    int64_t oct[G];
    int32_t nb[G][27];
    uint32_t sm[G][7];          // son masks: own, then sides x-, x+, y-, y+, z-, z+
    int32_t outside, coarse, split;   // some list entry outside the domain / a coarse cell; some son mask set
    int32_t live;                     // some cell is a leaf, or split cells are wanted too
    // the stencil's primitives are dead once the face states exist (phase
    // B), before the fluxes are written (phase C): one LDS region serves both
    union {
        R w[G][NV][kOctW];      // primitive variables of the stencil cells (planes, lds_get)
        double g[G][NV][kOctF]; // G = F dt/dx per face
    };
    union {
        R fs[G][2][NV][kOctF];      // face states: [0] left of the face, [1] right (planes)
        GhostCells<GH ? G * kOctGhosts : 0> ghost;   // before there are face states
    };
};

// GH: compiled with the interpolating coarse-ghost path; a.ghost then selects
// it.
// Bound like the sibling group (see hydro_sib) by the latency of its phases:
// table words, walls, split cells and coarse neighbours looked at only if the
// workgroup's octs have any, the update and the time step by the first wave.
template <typename R, int G, int NT, bool GH = false>
__device__ __forceinline__ void hydro_group(const LevelArgs &a, int64_t first, int count, Smem<R, G, GH> &S)
{
    static_assert(8 * G <= 64, "the own cells are updated by one wave");
    static_assert(G * kOctW <= 1024, "see GhostCells");
    const int tid = threadIdx.x;
    const double r = *a.dt / a.dx;
    const R h = static_cast<R>(0.5 * r);
    const R gam = static_cast<R>(a.gamma);
    const R g1 = static_cast<R>(1.0 / (a.gamma - 1.0));

    // oct indices, neighbour entries and son masks
    if (tid < G) S.oct[tid] = tid < count ? (a.list ? int64_t(a.list[first + tid]) : first + tid) : 0;
    if (tid == 0) {
        S.outside = S.coarse = S.split = 0;
        S.live = !a.skip_split;
        if constexpr (GH) S.ghost.n = 0;
    }
    __syncthreads();
    if (a.skip_split && tid < count && a.son[S.oct[tid]] != 0xffu) S.live = 1;
    for (int it = tid; it < count * 27; it += NT) {
        const int g = it / 27, s = it - 27 * g;
        const int32_t e = a.nbr27[27 * S.oct[g] + s];
        S.nb[g][s] = e;
        if (e < 0) (e == RG_NBR_OUTSIDE ? S.outside : S.coarse) = 1;
    }
    __syncthreads();
    // only split cells, which the restriction overwrites: nothing to do
    if (!S.live && !S.coarse) return;
    // by lanes of the last wave, put down after the gather
    uint32_t m = 0;
    const int ms = tid - (NT - 64), mg = ms / 7, mk = ms - 7 * mg;
    const bool mine = ms >= 0 && ms < 7 * count;
    if (mine) {
        int e = static_cast<int>(S.oct[mg]);
        if (mk) {
            const int ax = (mk - 1) >> 1, hi = (mk - 1) & 1, step = ax == 0 ? 1 : (ax == 1 ? 3 : 9);
            e = S.nb[mg][13 + (hi ? step : -step)];
        }
        if (e >= 0) m = a.son[e];
    }

    // A: gather uold for the stencil cells, primitive variables
    const bool outside = S.outside != 0;
    for (int it = tid; it < count * kOctW; it += NT) {
        const int g = it / kOctW, wc = it - kOctW * g;
        const uint32_t code = c_tab.wcode[wc];
        int entry = code & 31, bit = (code >> 5) & 7;
        if (outside) {
            int c[3], s[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                c[ax] = static_cast<int>((code >> (8 + 3 * ax)) & 7) - 2;
                s[ax] = slot_of(c[ax]);
            }
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
                if (s[ax] != 0 &&
                    S.nb[g][nslot(ax == 0 ? s[0] : 0, ax == 1 ? s[1] : 0, ax == 2 ? s[2] : 0)] == RG_NBR_OUTSIDE) {
                    c[ax] = s[ax] > 0 ? 1 : 0;
                    s[ax] = 0;
                }
            entry = nslot(s[0], s[1], s[2]);
            bit = (c[0] & 1) + 2 * (c[1] & 1) + 4 * (c[2] & 1);
        }
        int e = S.nb[g][entry];
        // a consistent list never leaves an outside slot here; an
        // inconsistent one reads the oct itself rather than stray memory
        if (e == RG_NBR_OUTSIDE) e = static_cast<int>(S.oct[g]);
        if constexpr (GH) {
            if (a.ghost && e < 0) {
                S.ghost.note(it, bit, e);
                continue;
            }
        }
        const double *src = e >= 0 ? a.uold + NV * (8 * int64_t(e) + bit) : a.ucoarse + NV * (-1 - int64_t(e));
        double U[NV], W[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) U[v] = src[v];
        prim64(U, a.gamma, W);
#pragma unroll
        for (int v = 0; v < NV; ++v) S.w[g][v][wc] = static_cast<R>(W[v]);
    }
    if constexpr (GH) {
        if (a.ghost && S.coarse) {
            __syncthreads();
            const int n = min(S.ghost.n, G * kOctGhosts);
            for (int k = tid; k < n * NV; k += NT) {
                const int i = k / NV, v = k - NV * i;
                S.ghost.u[v][i] = coarse_ghost(a, -1 - int64_t(S.ghost.coarse[i]), S.ghost.cell[i] >> 10, v);
            }
            __syncthreads();
            for (int i = tid; i < n; i += NT) {
                const int it = S.ghost.cell[i] & 1023, g = it / kOctW;
                double W[NV];
                prim64(ld5(S.ghost.u, i).v, a.gamma, W);
#pragma unroll
                for (int v = 0; v < NV; ++v) S.w[g][v][it - kOctW * g] = static_cast<R>(W[v]);
            }
        }
    }
    if (mine) {
        S.sm[mg][mk] = m;
        if (m) S.split = 1;
    }
    __syncthreads();

    // B: slopes, predictor and face states; the own cells of all octs first
    // (six states each), then the face-layer cells (one each)
    const bool split = S.split != 0;
    for (int it = tid; it < G * 32; it += NT) {
        const bool layer = it >= 8 * G;
        const int g = layer ? (it - 8 * G) / 24 : it >> 3;
        const int rc = layer ? it - 8 * G - 24 * g + 8 : it & 7;
        if (g >= count) continue;
        const uint64_t code = c_tab.rcode[rc];
        R dW[3][NV], Wp[NV], st[NV];
        reconstruct<R>(ld5(S.w[g], rc).v, ld5(S.w[g], code & 127).v, ld5(S.w[g], (code >> 7) & 127).v,
                       ld5(S.w[g], (code >> 14) & 127).v, ld5(S.w[g], (code >> 21) & 127).v,
                       ld5(S.w[g], (code >> 28) & 127).v, ld5(S.w[g], (code >> 35) & 127).v, h, gam, dW, Wp);
        if (!layer) {
            const int x = rc & 1, y = (rc >> 1) & 1, z = rc >> 2;
            const int f[3] = {face_id(0, x, y, z), face_id(1, y, x, z), face_id(2, z, x, y)};
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                face_state<R>(Wp, dW[ax], false, st);
                lds_put(S.fs[g][1], f[ax], st);
                face_state<R>(Wp, dW[ax], true, st);
                lds_put(S.fs[g][0], f[ax] + 4, st);
            }
        } else {
            const int fc = c_tab.fcode[rc - 8];
            const int side = (fc >> 6) & 1, ax = fc >> 7;
            R d[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) d[v] = ax == 0 ? dW[0][v] : (ax == 1 ? dW[1][v] : dW[2][v]);
            face_state<R>(Wp, d, side == 0, st);
            R *to = &S.fs[g][0][0][0] + side * (NV * kOctF) + (fc & 63);
#pragma unroll
            for (int v = 0; v < NV; ++v) to[v * kOctF] = st[v];
        }
    }
    __syncthreads();

    // C: HLLC on the 36 faces
    for (int it = tid; it < count * kOctF; it += NT) {
        const int g = it / kOctF, f = it - kOctF * g;
        const int ax = f >= 24 ? 2 : (f >= 12 ? 1 : 0);
        R L[NV], Rr[NV];
        lds_get(L, S.fs[g][0], f);
        lds_get(Rr, S.fs[g][1], f);
        bool zero = false;
        if (split) {
            // the two cells: position c-1 and c along the axis
            const int c = (f - 12 * ax) >> 2, t1 = f & 1, t2 = (f >> 1) & 1;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int pa = c - 1 + k;
                // cell position (pa along the axis, t1 / t2 across it) without a
                // run-time-indexed array, which would live in scratch memory
                const int px0 = ax == 0 ? pa : t1;
                const int px1 = ax == 1 ? pa : (ax == 0 ? t1 : t2);
                const int px2 = ax == 2 ? pa : t2;
                const int bit = (px0 & 1) + 2 * (px1 & 1) + 4 * (px2 & 1);
                const uint32_t sm = pa < 0 ? S.sm[g][1 + 2 * ax] : (pa > 1 ? S.sm[g][2 + 2 * ax] : S.sm[g][0]);
                zero = zero || ((sm >> bit) & 1u);
            }
        }
        double gf[NV];
        face_flux<R>(L, Rr, ax, gam, g1, r, zero, gf);
        lds_put(S.g[g], f, gf);
    }
    // the own cells are the first wave's to update; their old state is on its
    // way while the last faces are solved
    const int og = tid >> 3, oc = tid & 7;
    const bool owner = tid < 8 * G && og < count;
    double U[NV];
    int64_t own = 0;
    if (owner) {
        own = 8 * S.oct[og] + oc;
#pragma unroll
        for (int v = 0; v < NV; ++v) U[v] = a.uold[NV * own + v];
    }
    __syncthreads();

    // D: update and, fused, the CFL limit of the new state over the leaf cells
    // that no coarse-fine correction will change (no split face neighbour)
    if (tid < 64) {
        double best = __longlong_as_double(0x7ff0000000000000ll);
        double nf = 0.0;
        if (owner) {
            const int x = oc & 1, y = (oc >> 1) & 1, z = oc >> 2;
            const int fx = face_id(0, x, y, z), fy = face_id(1, y, x, z), fz = face_id(2, z, x, y);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const double *g = S.g[og][v];
                U[v] = ((U[v] + (g[fx] - g[fx + 4])) + (g[fy] - g[fy + 4])) + (g[fz] - g[fz + 4]);
                a.unew[NV * own + v] = U[v];
            }
            bool take = a.dt_next != nullptr;
            if (split) {
                const uint32_t m0 = S.sm[og][0];
                take = take && !((m0 >> oc) & 1u);
#pragma unroll
                for (int side = 0; side < 6; ++side) {
                    const int ax = side >> 1, hi = side & 1;
                    const uint32_t sm = ((oc >> ax) & 1) == hi ? S.sm[og][1 + side] : m0;
                    take = take && !((sm >> (oc ^ (1 << ax))) & 1u);
                }
            }
            if (take) {
                double W[NV];
                prim64(U, a.gamma, W);
                const double cs = sqrt_pos(div_pos(a.gamma * W[4], W[0]));
                const double sp = ((fabs(W[1]) + fabs(W[2])) + fabs(W[3])) + 3.0 * cs;
                const double cd = a.cfl * (a.dx / sp);
                best = cd < best ? cd : best;
                track_finite(nf, sp, U);
            }
        }
        if (a.dt_next) {
            best = nonfinite_limit(best, nf);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double o = __shfl_xor(best, off, 64);
                best = o < best ? o : best;
            }
            if (tid == 0) fold_min(a.dt_next, best, a.hdr);
        }
    } else if (S.coarse) {
        // E: flux owed to coarse neighbours, by the other waves.  Without a
        // buffer there must be none: a coarse face neighbour is then reported
        // (its flux is lost).
        for (int it = tid - 64; it < count * 6 * NV; it += NT - 64) {
            const int g = it / (6 * NV), k = it - 6 * NV * g;
            const int side = k / NV, v = k - NV * side;
            const int ax = side >> 1, hi = side & 1, step = ax == 0 ? 1 : (ax == 1 ? 3 : 9);
            const int e = S.nb[g][13 + (hi ? step : -step)];
            if (!(e < 0 && e != RG_NBR_OUTSIDE)) continue;
            if (!a.corr) {
                if (v == 0) flag_error(a.hdr, RG_EINVAL, S.oct[g]);
                continue;
            }
            const double *f = S.g[g][v] + face_id(ax, hi ? 2 : 0, 0, 0);
            const double sum = (f[0] + f[1]) + (f[2] + f[3]);
            const double d = 0.125 * sum;
            const double val = hi ? d : -d;
            double *dst = a.corr + 30 * (S.oct[g] - a.corr_base) + k;
            *dst = a.corr_mode == 0 ? val : (a.corr_mode == 1 ? 0.0 : *dst) + val;
        }
    }
}

}  // namespace
}  // namespace rg
