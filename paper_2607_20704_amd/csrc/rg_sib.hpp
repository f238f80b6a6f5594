// rg_sib.hpp -- hydro update of one complete sibling group: the 8 octs of
// one father oct, 4x4x4 cells, on one shared tile.
//
// Paper Sec. 3: grouping octs (nsubgrid) lets neighbouring octs share their
// stencil instead of each gathering its own ghost cells.  In a cell-by-cell
// tree the smallest such group that always exists wherever a cell is split
// is the set of its 8 children; outside the 8^3-oct bricks most octs belong
// to complete groups.  A group's tile spans cell offsets -2..5 per axis
// (relative to the group's low corner) and holds 304 cells (the 64 own
// cells, 96 in the face layer, 96 in the outer layer, 48 along the edges)
// against 8 x 80 for eight per-oct tiles; 160 cells are reconstructed (8 x
// 32 per oct) and 240 faces solved (8 x 36).  Each cell of the tile is
// reached through the neighbour list of the sibling whose own 6^3 tile holds
// it, with the same outside and coarse-ghost rules, and every value is
// formed by the same operations as in the per-oct body, so the two give the
// same bits.
#pragma once

#include "rg_oct.hpp"

namespace rg {
namespace {

constexpr int kSibW = 304;   // stencil cells
constexpr int kSibR = 160;   // reconstructed cells: own, then face layer
constexpr int kSibF = 240;   // faces: 3 axes x 5 planes x 16

// One word (or two) per item.  Own cells come first, x + 4y + 16z: the lanes
// of a wave then read neighbours in consecutive words (sibling by sibling, as
// in memory, they met in the same LDS banks four at a time).
struct SibTables {
    // stencil cell: list entry 27 sib + slot (8 bits), cell within that oct
    // (3), sibling whose 6^3 tile holds it (3), position in that tile + 2 (3
    // bits per axis)
    uint32_t wcode[kSibW];
    // reconstructed cell: its neighbours' indices x-, x+, y-, y+, z-, z+
    // (9 bits each)
    uint64_t rcode[kSibR];
    // face-layer cell: the face it has a state for (8 bits), which side of it
    // the state is (0 left, 1 right), axis (2 bits)
    uint16_t fcode[kSibR - 64];
};

constexpr int sib_tile(int x, int y, int z) { return (x + 2) + 8 * (y + 2) + 64 * (z + 2); }

// place 0 or 1 of the sibling whose 6^3 tile (cells -2..3 around its own
// two) covers group position p along one axis
constexpr int sib_place(int p) { return p < 0 ? 0 : (p > 3 ? 1 : p >> 1); }

// face on axis a between cells c-1 and c (c = 0..4) along a, at (t1, t2) on
// the other two axes in increasing order; bit 3 of the place is flipped on
// the planes c = 2, 3, which puts the faces of 32 consecutive cells in 32
// different double words of the LDS banks for every axis
__host__ __device__ constexpr int sib_face(int a, int c, int t1, int t2)
{
    return 80 * a + 16 * c + ((t1 + 4 * t2) ^ ((c & 2) << 2));
}

constexpr SibTables make_sib_tables()
{
    SibTables t{};
    int pos[kSibW][3] = {};
    int16_t index[512] = {};
    int n = 0;
    for (; n < 64; ++n)
        for (int a = 0; a < 3; ++a) pos[n][a] = (n >> (2 * a)) & 3;
    // face layer (reconstructed), then outer layer, per axis and side
    for (int layer = 0; layer < 2; ++layer)
        for (int a = 0; a < 3; ++a)
            for (int side = 0; side < 2; ++side)
                for (int q = 0; q < 16; ++q, ++n) {
                    const int t1 = a == 0 ? 1 : 0, t2 = a == 2 ? 1 : 2;
                    pos[n][a] = layer == 0 ? (side ? 4 : -1) : (side ? 5 : -2);
                    pos[n][t1] = q & 3;
                    pos[n][t2] = q >> 2;
                    // the high-side state of a cell below is left of face 0,
                    // the low-side state of a cell above right of face 4
                    if (layer == 0)
                        t.fcode[n - 64] = static_cast<uint16_t>(sib_face(a, side ? 4 : 0, q & 3, q >> 2) | side << 8 |
                                                                a << 9);
                }
    // edges: two coordinates in {-1, 4}, the third in 0..3
    for (int a = 0; a < 3; ++a)
        for (int q = 0; q < 16; ++q, ++n) {
            const int u = a == 0 ? 1 : 0, v = a == 2 ? 1 : 2;
            pos[n][a] = q & 3;
            pos[n][u] = (q >> 2) & 1 ? 4 : -1;
            pos[n][v] = (q >> 3) & 1 ? 4 : -1;
        }
    for (int i = 0; i < kSibW; ++i) {
        index[sib_tile(pos[i][0], pos[i][1], pos[i][2])] = static_cast<int16_t>(i);
        int sib = 0, slot = 13, cell = 0, where = 0;
        for (int a = 0, step = 1; a < 3; ++a, step *= 3) {
            const int place = sib_place(pos[i][a]), c = pos[i][a] - 2 * place;
            sib |= place << a;
            slot += c < 0 ? -step : (c > 1 ? step : 0);
            cell |= (c & 1) << a;
            where |= (c + 2) << (3 * a);
        }
        t.wcode[i] = static_cast<uint32_t>((27 * sib + slot) | cell << 8 | sib << 11 | where << 14);
    }
    for (int i = 0; i < kSibR; ++i) {
        const int x = pos[i][0], y = pos[i][1], z = pos[i][2];
        const int nb[6] = {index[sib_tile(x - 1, y, z)], index[sib_tile(x + 1, y, z)], index[sib_tile(x, y - 1, z)],
                           index[sib_tile(x, y + 1, z)], index[sib_tile(x, y, z - 1)], index[sib_tile(x, y, z + 1)]};
        for (int k = 0; k < 6; ++k) t.rcode[i] |= static_cast<uint64_t>(nb[k]) << (9 * k);
    }
    return t;
}

__constant__ SibTables c_sib = make_sib_tables();

// neighbour-list slot of face side 2 * axis + high
__device__ __forceinline__ int side_slot(int ax, int hi)
{
    const int d = hi ? 1 : -1;
    return nslot(ax == 0 ? d : 0, ax == 1 ? d : 0, ax == 2 ? d : 0);
}

// Workgroup size: FP64 one stencil cell per thread, 69 registers: seven waves
// per SIMD, 28 on a compute unit, hold five workgroups (a sixth needs 30), and
// so does the LDS (32.4 KB each), so that easing one alone gains nothing; 256
// threads take 84 registers; mixed four waves, one per SIMD (clumps of levels
// 7-11, one step: FP64 830 us at 320 threads, 840 at 256; mixed 634 and 562;
// with interpolated ghosts FP64 947 and 966, mixed 719 and 662).
__host__ __device__ constexpr int sib_threads(bool fp64) { return fp64 ? 320 : 256; }

template <typename R, bool GH = false> struct SibSmem {
    int32_t oct[8];             // by place in the group
    int32_t nb[8 * 27];
    // son masks: [0, 8) the siblings; 8 + 4 side + q the neighbour across
    // side (2 axis + high) of the siblings on that face, q = their place
    // along the two other axes (lower axis first)
    uint32_t sm[32];
    int32_t outside, coarse, split;   // some list entry outside the domain / a coarse cell; some son mask set
    int32_t live;                     // some cell is a leaf, or split cells are wanted too
    // the primitives are dead once the face states exist
    union {
        R w[NV][kSibW];         // primitive variables of the stencil cells (planes, lds_get)
        double g[NV][kSibF];    // G = F dt/dx per face
    };
    union {
        R fs[2][NV][kSibF];         // face states: [0] left of the face, [1] right (planes)
        GhostCells<GH ? kSibW - 64 : 0> ghost;   // before there are face states
    };
};

// son mask holding the cell at group position (x, y, z), one coordinate of
// which may lie one cell outside the group
__device__ __forceinline__ uint32_t sib_mask_at(const uint32_t *sm, int x, int y, int z)
{
    if (x < 0) return sm[8 + 0 + (y >> 1) + 2 * (z >> 1)];
    if (x > 3) return sm[8 + 4 + (y >> 1) + 2 * (z >> 1)];
    if (y < 0) return sm[8 + 8 + (x >> 1) + 2 * (z >> 1)];
    if (y > 3) return sm[8 + 12 + (x >> 1) + 2 * (z >> 1)];
    if (z < 0) return sm[8 + 16 + (x >> 1) + 2 * (y >> 1)];
    if (z > 3) return sm[8 + 20 + (x >> 1) + 2 * (y >> 1)];
    return sm[(x >> 1) + 2 * (y >> 1) + 4 * (z >> 1)];
}

// What bounds it: latency and issue, not memory.  A group takes about 12 us
// from its first load to its last store, most of it waiting for dependent
// loads and barriers, and the chip holds as many groups as their LDS and
// registers allow.
// Of 3200 VALU instructions per FP64 group 1400 are the scheme's arithmetic;
// the rest was index arithmetic, three divergent passes over the axes for
// cells of the face layer, which have one state each, and tests for walls,
// split cells and coarse neighbours in groups that have none.  Those are
// decided once per group here, indices come from one table word per item, and
// the state is kept once.
template <typename R, int NT, bool GH>
__device__ __forceinline__ void hydro_sib(const LevelArgs &a, const int32_t *__restrict__ father, int64_t first,
                                          SibSmem<R, GH> &S)
{
    const int tid = threadIdx.x;
    const double r = *a.dt / a.dx;
    const R h = static_cast<R>(0.5 * r);
    const R gam = static_cast<R>(a.gamma);
    const R g1 = static_cast<R>(1.0 / (a.gamma - 1.0));

    // the siblings by place (the father cell's index in its oct), their
    // neighbour lists and son masks; the places of a consistent tree are a
    // permutation, and an inconsistent one still names octs of the group
    // lists of the group are read in key order together with the places they
    // belong to, not after them: one memory round trip less
    int32_t e0 = 0, f0 = 0;
    uint32_t m0 = 0xffu;
    static_assert(NT >= 8 * 27, "one thread per list entry");
    const int g0 = tid / 27, s0 = tid - 27 * g0;
    if (tid < 8 * 27) {
        e0 = a.nbr27[27 * first + tid];
        f0 = father[first + g0];
        if (s0 == 0 && a.skip_split) m0 = a.son[first + g0];
        S.nb[tid] = RG_NBR_OUTSIDE;
    }
    if (tid < 8) S.oct[tid] = static_cast<int32_t>(first) + tid;
    if (tid == 0) {
        S.outside = S.coarse = S.split = 0;
        S.live = !a.skip_split;
        if constexpr (GH) S.ghost.n = 0;
    }
    __syncthreads();
    if (tid < 8 * 27) {
        S.nb[27 * (f0 & 7) + s0] = e0;
        if (e0 < 0) (e0 == RG_NBR_OUTSIDE ? S.outside : S.coarse) = 1;
        if (s0 == 0) {
            S.oct[f0 & 7] = static_cast<int32_t>(first) + g0;
            if (m0 != 0xffu) S.live = 1;
        }
    }
    __syncthreads();
    // only split cells, which the restriction overwrites: nothing to do
    if (!S.live && !S.coarse) return;
    // son masks, by lanes of the last wave, put down after the gather
    uint32_t m = 0;
    const int ms = tid - (NT - 64);
    if (ms >= 0 && ms < 32) {
        int e;
        if (ms < 8) {
            e = S.oct[ms];
        } else {
            const int side = (ms - 8) >> 2, q = (ms - 8) & 3;
            const int ax = side >> 1, hi = side & 1;
            const int t1 = ax == 0 ? 1 : 0, t2 = ax == 2 ? 1 : 2;
            const int sib = (hi << ax) | ((q & 1) << t1) | ((q >> 1) << t2);
            e = S.nb[27 * sib + side_slot(ax, hi)];
        }
        if (e >= 0) m = a.son[e];
    }

    // A: gather uold for the stencil cells, primitive variables
    const bool outside = S.outside != 0;
    for (int it = tid; it < kSibW; it += NT) {
        const uint32_t code = c_sib.wcode[it];
        int entry = code & 255, bit = (code >> 8) & 7;
        const int sib = (code >> 11) & 7;
        if (outside) {
            int c[3], s[3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                c[ax] = static_cast<int>((code >> (14 + 3 * ax)) & 7) - 2;
                s[ax] = slot_of(c[ax]);
            }
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
                if (s[ax] != 0 &&
                    S.nb[27 * sib + nslot(ax == 0 ? s[0] : 0, ax == 1 ? s[1] : 0, ax == 2 ? s[2] : 0)] == RG_NBR_OUTSIDE) {
                    c[ax] = s[ax] > 0 ? 1 : 0;
                    s[ax] = 0;
                }
            entry = 27 * sib + nslot(s[0], s[1], s[2]);
            bit = (c[0] & 1) + 2 * (c[1] & 1) + 4 * (c[2] & 1);
        }
        int e = S.nb[entry];
        if (e == RG_NBR_OUTSIDE) e = S.oct[sib];
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
        for (int v = 0; v < NV; ++v) S.w[v][it] = static_cast<R>(W[v]);
    }
    if constexpr (GH) {
        if (a.ghost && S.coarse) {
            __syncthreads();
            const int n = min(S.ghost.n, kSibW - 64);
            for (int k = tid; k < n * NV; k += NT) {
                const int i = k / NV, v = k - NV * i;
                S.ghost.u[v][i] = coarse_ghost(a, -1 - int64_t(S.ghost.coarse[i]), S.ghost.cell[i] >> 10, v);
            }
            __syncthreads();
            for (int i = tid; i < n; i += NT) {
                double W[NV];
                prim64(ld5(S.ghost.u, i).v, a.gamma, W);
#pragma unroll
                for (int v = 0; v < NV; ++v) S.w[v][S.ghost.cell[i] & 1023] = static_cast<R>(W[v]);
            }
        }
    }
    if (ms >= 0 && ms < 32) {
        S.sm[ms] = m;
        if (m) S.split = 1;
    }
    __syncthreads();

    // B: slopes, predictor and face states of the own and face-layer cells
    const bool split = S.split != 0;
    for (int it = tid; it < kSibR; it += NT) {
        const uint64_t code = c_sib.rcode[it];
        R dW[3][NV], Wp[NV], st[NV];
        reconstruct<R>(ld5(S.w, it).v, ld5(S.w, code & 511).v, ld5(S.w, (code >> 9) & 511).v,
                       ld5(S.w, (code >> 18) & 511).v, ld5(S.w, (code >> 27) & 511).v, ld5(S.w, (code >> 36) & 511).v,
                       ld5(S.w, (code >> 45) & 511).v, h, gam, dW, Wp);
        if (it < 64) {
            const int x = it & 3, y = (it >> 2) & 3, z = it >> 4;
            const int lo[3] = {sib_face(0, x, y, z), sib_face(1, y, x, z), sib_face(2, z, x, y)};
            const int hi[3] = {sib_face(0, x + 1, y, z), sib_face(1, y + 1, x, z), sib_face(2, z + 1, x, y)};
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                face_state<R>(Wp, dW[ax], false, st);
                lds_put(S.fs[1], lo[ax], st);
                face_state<R>(Wp, dW[ax], true, st);
                lds_put(S.fs[0], hi[ax], st);
            }
        } else {
            const int fc = c_sib.fcode[it - 64];
            const int side = (fc >> 8) & 1, ax = fc >> 9;
            R d[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) d[v] = ax == 0 ? dW[0][v] : (ax == 1 ? dW[1][v] : dW[2][v]);
            face_state<R>(Wp, d, side == 0, st);
            R *to = &S.fs[0][0][0] + side * (NV * kSibF) + (fc & 255);
#pragma unroll
            for (int v = 0; v < NV; ++v) to[v * kSibF] = st[v];
        }
    }
    __syncthreads();

    // C: HLLC on the 240 faces
    for (int f = tid; f < kSibF; f += NT) {
        const int ax = f >= 160 ? 2 : (f >= 80 ? 1 : 0);
        R L[NV], Rr[NV];
        lds_get(L, S.fs[0], f);
        lds_get(Rr, S.fs[1], f);
        bool zero = false;
        if (split) {
            const int c = (f - 80 * ax) >> 4, t = (f & 15) ^ ((c & 2) << 2), t1 = t & 3, t2 = t >> 2;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int pa = c - 1 + k;
                const int px0 = ax == 0 ? pa : t1;
                const int px1 = ax == 1 ? pa : (ax == 0 ? t1 : t2);
                const int px2 = ax == 2 ? pa : t2;
                const int bit = (px0 & 1) + 2 * (px1 & 1) + 4 * (px2 & 1);
                zero = zero || ((sib_mask_at(S.sm, px0, px1, px2) >> bit) & 1u);
            }
        }
        double gf[NV];
        face_flux<R>(L, Rr, ax, gam, g1, r, zero, gf);
        lds_put(S.g, f, gf);
    }
    // the own cells are the first wave's to update; their old state is on its
    // way while the last faces are solved
    const int x = tid & 3, y = (tid >> 2) & 3, z = (tid >> 4) & 3;
    const int own_sib = (x >> 1) + 2 * (y >> 1) + 4 * (z >> 1), own_bit = (x & 1) + 2 * (y & 1) + 4 * (z & 1);
    double U[NV];
    int64_t own = 0;
    if (tid < 64) {
        own = 8 * int64_t(S.oct[own_sib]) + own_bit;
#pragma unroll
        for (int v = 0; v < NV; ++v) U[v] = a.uold[NV * own + v];
    }
    __syncthreads();

    // D: update and, fused, the CFL limit of the new state over the leaf cells
    // that no coarse-fine correction will change (no split face neighbour)
    if (tid < 64) {
        const int fx = sib_face(0, x, y, z), fy = sib_face(1, y, x, z), fz = sib_face(2, z, x, y);
        const int gx = sib_face(0, x + 1, y, z), gy = sib_face(1, y + 1, x, z), gz = sib_face(2, z + 1, x, y);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double *g = S.g[v];
            U[v] = ((U[v] + (g[fx] - g[gx])) + (g[fy] - g[gy])) + (g[fz] - g[gz]);
            a.unew[NV * own + v] = U[v];
        }
        if (a.dt_next) {
            double best = __longlong_as_double(0x7ff0000000000000ll);
            double nf = 0.0;
            bool take = true;
            if (split) {
                take = !((S.sm[own_sib] >> own_bit) & 1u);
#pragma unroll
                for (int side = 0; side < 6; ++side) {
                    const int ax = side >> 1, d = (side & 1) ? 1 : -1;
                    const int px = x + (ax == 0 ? d : 0), py = y + (ax == 1 ? d : 0), pz = z + (ax == 2 ? d : 0);
                    take = take && !((sib_mask_at(S.sm, px, py, pz) >> (own_bit ^ (1 << ax))) & 1u);
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
            best = nonfinite_limit(best, nf);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double o = __shfl_xor(best, off, 64);
                best = o < best ? o : best;
            }
            if (tid == 0) fold_min(a.dt_next, best, a.hdr);
        }
    } else if (S.coarse) {
        // E: flux owed to coarse neighbours across the group's outer faces, by
        // the other waves; without a buffer there must be none (a coarse
        // neighbour is reported)
        for (int it = tid - 64; it < 8 * 3 * NV; it += NT - 64) {
            const int p = it / NV, v = it - NV * p;
            const int sib = p / 3, ax = p - 3 * sib, hi = (sib >> ax) & 1;
            const int e = S.nb[27 * sib + side_slot(ax, hi)];
            if (!(e < 0 && e != RG_NBR_OUTSIDE)) continue;
            if (!a.corr) {
                if (v == 0) flag_error(a.hdr, RG_EINVAL, S.oct[sib]);
                continue;
            }
            const int t1 = ax == 0 ? 1 : 0, t2 = ax == 2 ? 1 : 2;
            const int f = sib_face(ax, hi ? 4 : 0, 2 * ((sib >> t1) & 1), 2 * ((sib >> t2) & 1));
            const double sum = (S.g[v][f] + S.g[v][f + 1]) + (S.g[v][f + 4] + S.g[v][f + 5]);
            const double d = 0.125 * sum;
            const double val = hi ? d : -d;
            double *dst = a.corr + 30 * (S.oct[sib] - a.corr_base) + NV * (2 * ax + hi) + v;
            *dst = a.corr_mode == 0 ? val : (a.corr_mode == 1 ? 0.0 : *dst) + val;
        }
    }
}

}  // namespace
}  // namespace rg
