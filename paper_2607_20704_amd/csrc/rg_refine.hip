// rg_refine.hip -- refinement and de-refinement of the oct tree on the device.
//
// Paper Sec. 2.2: every step the tree changes in four stages: new octs under
// flagged cells, removal of the children of split cells that are no longer
// flagged, a bucket sort by level and a Hilbert sort inside each level.  No
// sort is needed here: the new tree's octs of a level are the children of the
// old tree's octs of the level above (every flagged cell has one), in those
// octs' order and along the curve inside each, so a prefix over the old octs
// of the number of flagged cells gives every new oct its place.  The paper
// does not give the criterion or the grading rule; the ones used (density
// threshold or density jump across a face; a flagged cell needs its 26
// neighbours at its own level, which flags the coarser cells under them,
// finest level first) are restated in the header next to rg_refine.
//
// Everything runs on the device with the tree's own neighbour lists: the
// criterion reads the six face neighbours through the 27-entry list, the
// closure marks father cells through it (a missing neighbour oct's entry is
// already the coarse cell under it), and the new oct list comes from a prefix
// over per-oct counts, whose values at the old level boundaries are the new
// level ranges: the one thing the host reads back.
#include "rg_compact.hpp"
#include "rg_internal.hpp"

namespace rg {

size_t nbr_lists_ws_bytes(int64_t n);
rg_status nbr_lists_device(const uint64_t *d_keys, int64_t n, const int64_t *h_level_begin, int lmin, int lmax,
                           void *d_ws, size_t ws_bytes, const int32_t **list, const uint32_t **d_count, hipStream_t s);

namespace {

constexpr int NVR = 5;   // conserved variables per cell

__device__ __forceinline__ int face_slot(int side)
{
    // x-, x+, y-, y+, z-, z+ in the (dx+1) + 3(dy+1) + 9(dz+1) numbering
    return side == 0 ? 12 : side == 1 ? 14 : side == 2 ? 10 : side == 3 ? 16 : side == 4 ? 4 : 22;
}

struct CritArgs {
    const double *u;
    const int32_t *nbr27;
    int64_t ob, oe;       // octs of the levels that may be flagged
    double rho_thresh, grad_thresh;
    uint32_t *flags;
    int whole;            // widen a flag to all 8 cells of its oct (4^3-cell blocks)
};

// one thread per cell: the criterion on the cell's density and its six face
// neighbours' (same-level cell, else the coarse cell under the missing oct,
// outside: the cell itself).  Launched with a multiple of 64 threads per
// block, so an oct's eight cells sit in one wave.
__global__ void k_refine_criterion(CritArgs a)
{
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t o = a.ob + (t >> 3);
    if (o >= a.oe) return;
    const int c = static_cast<int>(t & 7);
    const int cx = c & 1, cy = (c >> 1) & 1, cz = c >> 2;
    const double rc = a.u[NVR * (8 * o + c)];
    bool flag = a.rho_thresh > 0.0 && rc > a.rho_thresh;
    if (a.grad_thresh > 0.0) {
        for (int side = 0; side < 6; ++side) {
            int p[3] = {cx, cy, cz};
            const int ax = side >> 1;
            p[ax] += (side & 1) ? 1 : -1;
            double rn;
            if (p[ax] >= 0 && p[ax] <= 1) {
                rn = a.u[NVR * (8 * o + p[0] + 2 * p[1] + 4 * p[2])];
            } else {
                const int32_t e = a.nbr27[27 * o + face_slot(side)];
                if (e == RG_NBR_OUTSIDE) {
                    rn = rc;
                } else if (e >= 0) {
                    const int q[3] = {p[0] & 1, p[1] & 1, p[2] & 1};
                    rn = a.u[NVR * (8 * int64_t(e) + q[0] + 2 * q[1] + 4 * q[2])];
                } else {
                    rn = a.u[NVR * (-1 - int64_t(e))];
                }
            }
            const double d = fabs(rn - rc) / (rn + rc);
            flag = flag || d > a.grad_thresh;
        }
    }
    // the eight lanes of an oct are eight consecutive lanes of one wave
    const uint64_t votes = __ballot(flag);
    const int lane = threadIdx.x & 63;
    uint32_t m = static_cast<uint32_t>((votes >> (lane & ~7)) & 0xffu);
    if (a.whole && m) m = 0xffu;
    if (c == 0) a.flags[o] = m;
}

__global__ void k_zero_u32(uint32_t *p, int64_t n)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// 32 lanes per oct of one level (27 used): a flagged cell marks the father
// cell of every level-l oct holding one of its 26 neighbours or itself.  A
// cell with in-oct position c reaches, along each axis, its own oct and the
// neighbour oct on its side (offset -1 for c = 0, +1 for c = 1): the oct's
// list entry at offset d is needed if a flagged cell lies on d's side along
// every axis where d is not zero.  Each lane takes one entry, so that an oct
// costs one chain of loads (one thread per oct went through up to 27 of them:
// 25 us a level); each target bit is set by an atomic only if a plain read
// does not already show it (many octs mark the same coarse cells).
__global__ void k_refine_closure(const int32_t *__restrict__ nbr27, const int32_t *__restrict__ father,
                                 int64_t ob, int64_t oe, uint32_t *flags, int whole)
{
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t o = ob + (t >> 5);
    const int slot = static_cast<int>(t & 31);
    if (o >= oe || slot >= 27) return;
    const uint32_t m = flags[o] & 0xffu;
    if (!m) return;
    const int s[3] = {slot % 3 - 1, (slot / 3) % 3 - 1, slot / 9 - 1};
    constexpr uint32_t high[3] = {0xaau, 0xccu, 0xf0u};   // cells on the high side of each axis
    uint32_t reach = 0xffu;
#pragma unroll
    for (int a = 0; a < 3; ++a) reach &= s[a] > 0 ? high[a] : (s[a] < 0 ? ~high[a] : 0xffu);
    if (!(m & reach)) return;
    const int32_t e = nbr27[27 * o + slot];
    if (e == RG_NBR_OUTSIDE) return;
    const int64_t fc = e >= 0 ? int64_t(father[e]) : (-1 - int64_t(e));
    if (fc < 0) return;   // coarsest level: nothing to mark
    const uint32_t bit = whole ? 0xffu : 1u << (fc & 7);
    if ((flags[fc >> 3] & bit) != bit) atomicOr(&flags[fc >> 3], bit);
}

__device__ __forceinline__ bool kept(const uint32_t *flags, const int32_t *father, int64_t o, bool coarsest)
{
    if (coarsest) return true;
    const int32_t f = father[o];
    return f >= 0 && ((flags[f >> 3] >> (f & 7)) & 1u);
}

// children of old oct o in the new tree
__device__ __forceinline__ uint32_t children(const uint32_t *flags, const int32_t *father, int64_t o, int64_t coarse_end)
{
    return kept(flags, father, o, o < coarse_end) ? static_cast<uint32_t>(__popc(flags[o] & 0xffu)) : 0u;
}

__global__ __launch_bounds__(kItems) void k_refine_count(const uint32_t *__restrict__ flags,
                                                         const int32_t *__restrict__ father, int64_t n,
                                                         int64_t coarse_end, uint32_t *__restrict__ cnt)
{
    __shared__ uint32_t s[kItems / 64];
    const int64_t o = int64_t(blockIdx.x) * kItems + threadIdx.x;
    uint32_t total;
    (void)block_prefix(o < n ? children(flags, father, o, coarse_end) : 0u, s, total);
    if (threadIdx.x == 0) cnt[blockIdx.x] = total;
}

// off[o]: children of the octs before o; bound[j]: of those before marks.at[j]
__global__ __launch_bounds__(kItems) void k_refine_offsets(const uint32_t *__restrict__ flags,
                                                           const int32_t *__restrict__ father, int64_t n,
                                                           int64_t coarse_end, const uint32_t *__restrict__ cnt,
                                                           const uint32_t *__restrict__ all, Marks marks,
                                                           uint32_t *__restrict__ off, int64_t *__restrict__ bound)
{
    __shared__ uint32_t s[kItems / 64];
    const int64_t o = int64_t(blockIdx.x) * kItems + threadIdx.x;
    uint32_t total;
    const uint32_t first = cnt[blockIdx.x];
    const uint32_t p = block_prefix(o < n ? children(flags, father, o, coarse_end) : 0u, s, total);
    __shared__ uint32_t before[kItems];
    before[threadIdx.x] = p;
    if (o < n) off[o] = first + p;
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < marks.n) {
        const int64_t at = marks.at[threadIdx.x], q = at - int64_t(blockIdx.x) * kItems;
        if (at >= n) {
            if (blockIdx.x == 0) bound[threadIdx.x] = *all;
        } else if (q >= 0 && q < kItems) {
            bound[threadIdx.x] = first + before[q];
        }
    }
}

// The eight cells of the oct with key K along the curve: the cell at place h
// is c0 ^ (the Gray code of h with its three bits sent to a, b, c), so the
// first three places give the rest.  K << 3 | h is the key of the child oct
// under that cell, whose coordinates' low bits are the cell.
struct CurveCells {
    int c0, a, b, c;

    __device__ __forceinline__ explicit CurveCells(uint64_t K)
    {
        int v[3];
#pragma unroll
        for (int h = 0; h < 3; ++h) {
            int32_t i, j, k, l;
            key_coords((K << 3) | uint64_t(h), i, j, k, l);
            v[h] = (i & 1) + 2 * (j & 1) + 4 * (k & 1);
        }
        c0 = v[0];
        a = v[0] ^ v[1];
        b = v[1] ^ v[2];
        c = 7 ^ a ^ b;
    }

    __device__ __forceinline__ int cell(int h) const
    {
        const int g = h ^ (h >> 1);
        return c0 ^ ((g & 1) ? a : 0) ^ ((g & 2) ? b : 0) ^ ((g & 4) ? c : 0);
    }
};

struct EmitArgs {
    const uint32_t *flags, *son, *off;
    const int32_t *father, *ijkl;
    const uint64_t *keys;
    int64_t n, coarse_end, cap;
    int32_t *src, *new_ijkl;
    uint64_t *new_keys;
};

// new oct p: its source (an old oct, or -1 - the cell it is under), key and
// coordinates; places past the capacity are left out
__device__ __forceinline__ void emit(const EmitArgs &a, int64_t p, int32_t src, uint64_t key, int i, int j, int k, int l)
{
    if (p >= a.cap) return;
    a.src[p] = src;
    a.new_keys[p] = key;
    reinterpret_cast<int4 *>(a.new_ijkl)[p] = make_int4(i, j, k, l);
}

// every old oct: its own new place, if it is kept, and the new children under
// its flagged leaf cells.  The coarsest level comes first and is kept whole.
__global__ __launch_bounds__(256) void k_refine_emit(EmitArgs a)
{
    const int64_t o = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (o >= a.n) return;
    if (!kept(a.flags, a.father, o, o < a.coarse_end)) return;
    const uint64_t K = a.keys[o];
    const int32_t i = a.ijkl[4 * o], j = a.ijkl[4 * o + 1], k = a.ijkl[4 * o + 2], l = a.ijkl[4 * o + 3];
    int64_t p = o;
    if (o >= a.coarse_end) {
        // place among the father's flagged cells
        const int64_t f = a.father[o] >> 3;
        const uint32_t m = a.flags[f] & 0xffu;
        const int h = static_cast<int>(K & 7);
        int rank = h;
        if (m != 0xffu) {
            const CurveCells cells(K >> 3);
            rank = 0;
            for (int g = 0; g < h; ++g) rank += (m >> cells.cell(g)) & 1;
        }
        p = a.coarse_end + a.off[f] + rank;
    }
    emit(a, p, static_cast<int32_t>(o), K, i, j, k, l);
    const uint32_t m = a.flags[o] & 0xffu;
    if (!(m & ~a.son[o])) return;
    const CurveCells cells(K);
    int64_t q = a.coarse_end + a.off[o];
    for (int h = 0; h < 8; ++h) {
        const int c = cells.cell(h);
        if (!((m >> c) & 1u)) continue;
        if (!((a.son[o] >> c) & 1u))
            emit(a, q, static_cast<int32_t>(-1 - (8 * o + c)), (K << 3) | uint64_t(h), 2 * i + (c & 1),
                 2 * j + ((c >> 1) & 1), 2 * k + (c >> 2), l + 1);
        ++q;
    }
}

// new oct p: key, coordinates and state; a kept oct copies its 8 cells, a new
// one repeats its father cell.  V: doubles per load and store (2 where both
// states and the coordinates are 16-byte aligned).  The copy of the state is
// what bounds it.
template <int V>
__global__ __launch_bounds__(256) void k_refine_gather(const int32_t *__restrict__ new_ijkl,
                                                       const uint64_t *__restrict__ new_keys,
                                                       const int32_t *__restrict__ src, const double *__restrict__ u,
                                                       int64_t n, int64_t m, int32_t *__restrict__ ijkl_out,
                                                       uint64_t *__restrict__ keys_out, double *__restrict__ u_out)
{
    constexpr int T = 40 / V;   // threads per oct
    const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const int64_t p = t / T;
    const int r = static_cast<int>(t - T * p);
    if (p >= m) return;
    // son masks and father cells that contradict each other leave places
    // without a source: those read the first oct
    int32_t s = src[p];
    if (s >= n || -1 - int64_t(s) >= 8 * n) s = 0;
    if (r == 0) keys_out[p] = new_keys[p];
    if constexpr (V == 2) {
        if (r == 1) reinterpret_cast<int4 *>(ijkl_out)[p] = reinterpret_cast<const int4 *>(new_ijkl)[p];
        double2 v;
        if (s >= 0) {
            v = reinterpret_cast<const double2 *>(u + 40 * int64_t(s))[r];
        } else {
            const double *c = u + NVR * (-1 - int64_t(s));
            v.x = c[(2 * r) % NVR];
            v.y = c[(2 * r + 1) % NVR];
        }
        reinterpret_cast<double2 *>(u_out + 40 * p)[r] = v;
    } else {
        if (r < 4) ijkl_out[4 * p + r] = new_ijkl[4 * p + r];
        u_out[40 * p + r] = s >= 0 ? u[40 * int64_t(s) + r] : u[NVR * (-1 - int64_t(s)) + (r % NVR)];
    }
}

__global__ void k_refine_levels(int64_t *begin, Marks lb)
{
    if (threadIdx.x < RG_MAX_LEVEL + 2) begin[threadIdx.x] = lb.at[threadIdx.x];
}

struct RefineWs {
    uint32_t *flags, *off, *cnt, *total;
    int32_t *src, *new_ijkl;
    int64_t *bound;
};

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

size_t core_bytes(int64_t cap)
{
    return 3 * al256(4 * cap) + al256(16 * cap) + al256(4 * item_blocks(cap)) + 512;
}

RefineWs carve(void *ws, int64_t cap)
{
    char *p = static_cast<char *>(ws);
    RefineWs w;
    w.total = reinterpret_cast<uint32_t *>(p);
    p += 256;
    w.bound = reinterpret_cast<int64_t *>(p);
    p += 256;
    w.flags = reinterpret_cast<uint32_t *>(p);
    p += al256(4 * cap);
    w.off = reinterpret_cast<uint32_t *>(p);
    p += al256(4 * cap);
    w.src = reinterpret_cast<int32_t *>(p);
    p += al256(4 * cap);
    w.new_ijkl = reinterpret_cast<int32_t *>(p);
    p += al256(16 * cap);
    w.cnt = reinterpret_cast<uint32_t *>(p);
    return w;
}

rg_status check_tree(const rg_tree *t, const rg_refine_params *pr)
{
    RG_REQUIRE(t && pr, "null pointer");
    RG_REQUIRE(t->n_oct > 0 && t->lmin >= 1 && t->lmax >= t->lmin && t->lmax <= RG_MAX_LEVEL, "bad tree");
    RG_REQUIRE(t->level_begin[t->lmin] == 0 && t->level_begin[t->lmax + 1] == t->n_oct, "bad level ranges");
    RG_REQUIRE(t->d_nbr27 && t->d_father_cell && t->d_son_mask, "tree without neighbour lists");
    RG_REQUIRE(pr->lmax >= t->lmin && pr->lmax <= RG_MAX_LEVEL, "refinement level limit %d out of range", pr->lmax);
    RG_REQUIRE(pr->nsubgrid == 0 || pr->nsubgrid == 2 || pr->nsubgrid == 4, "nsubgrid %d not 2 or 4", pr->nsubgrid);
    return RG_OK;
}

// criterion, then (if closure) the grading closure from the finest level down
rg_status flags_pass(const rg_tree *t, const double *d_u, const rg_refine_params *pr, int closure, uint32_t *flags,
                     hipStream_t s)
{
    k_zero_u32<<<grid_for(t->n_oct, 256), 256, 0, s>>>(flags, t->n_oct);
    RG_TRY(launch_status("refine flags clear"));
    const int ltop = t->lmax < pr->lmax - 1 ? t->lmax : pr->lmax - 1;
    if (ltop >= t->lmin) {
        CritArgs a;
        a.u = d_u;
        a.nbr27 = t->d_nbr27;
        a.ob = 0;
        a.oe = t->level_begin[ltop + 1];
        a.rho_thresh = pr->rho_thresh;
        a.grad_thresh = pr->grad_thresh;
        a.flags = flags;
        a.whole = pr->nsubgrid == 4;
        if (a.oe > 0) {
            k_refine_criterion<<<grid_for(8 * a.oe, 256), 256, 0, s>>>(a);
            RG_TRY(launch_status("refine criterion"));
        }
    }
    if (closure) {
        // no cell above ltop is flagged
        for (int l = ltop; l > t->lmin; --l) {
            const int64_t ob = t->level_begin[l], oe = t->level_begin[l + 1];
            if (oe <= ob) continue;
            k_refine_closure<<<grid_for(32 * (oe - ob), 256), 256, 0, s>>>(t->d_nbr27, t->d_father_cell, ob, oe, flags,
                                                                    pr->nsubgrid == 4);
            RG_TRY(launch_status("refine closure"));
        }
    }
    return RG_OK;
}

}  // namespace
}  // namespace rg

using namespace rg;

extern "C" {

size_t rg_refine_workspace_bytes(int64_t capacity)
{
    const int64_t cap = capacity > 0 ? capacity : 1;
    return core_bytes(cap) + al256(nbr_lists_ws_bytes(cap));
}

rg_status rg_refine_flags(const rg_tree *t, const double *d_u, const rg_refine_params *p, int closure,
                          uint32_t *d_flags, void *stream)
{
    RG_TRY(check_tree(t, p));
    RG_REQUIRE(d_u && d_flags, "null pointer");
    return flags_pass(t, d_u, p, closure, d_flags, as_stream(stream));
}

rg_status rg_refine(rg_tree *t, const double *d_u, double *d_u_new, const rg_refine_params *p, void *d_ws,
                    size_t ws_bytes, void *stream)
{
    RG_TRY(check_tree(t, p));
    RG_REQUIRE(d_u && d_u_new && d_ws, "null pointer");
    RG_REQUIRE(d_u != d_u_new, "state buffers must not alias");
    RG_REQUIRE(t->d_ijkl && t->d_keys_scratch && t->d_perm && t->d_sort_ws && t->d_level_begin && t->d_hash_ws,
               "refinement needs coordinates, scratch keys, permutation, sort workspace, level ranges and hash "
               "workspace");
    const int64_t cap = t->capacity > 0 ? t->capacity : t->n_oct;
    RG_REQUIRE(cap >= t->n_oct && cap <= (int64_t(1) << 28), "capacity %lld below the oct count",
               static_cast<long long>(cap));
    RG_REQUIRE(ws_bytes >= rg_refine_workspace_bytes(cap) && aligned(d_ws, 256), "refine workspace too small");
    RG_REQUIRE(t->sort_ws_bytes >= rg_sort_workspace_bytes(cap), "sort workspace below capacity");
    RG_REQUIRE(t->hash_ws_bytes >= rg_hash_workspace_bytes(cap), "hash workspace below capacity");
    // the old tree's keys are read and the new ones formed in the scratch
    // keys before they are copied over them
    RG_REQUIRE(t->d_keys && t->d_keys != t->d_keys_scratch, "refinement needs keys, and scratch keys apart from them");
    RG_REQUIRE(aligned(t->d_keys, 8) && aligned(t->d_keys_scratch, 8), "misaligned keys");
    RG_REQUIRE(aligned(t->d_sort_ws, 256) && aligned(t->d_hash_ws, 256), "workspaces must be 256-byte aligned");
    hipStream_t s = as_stream(stream);
    const int64_t n = t->n_oct;
    RefineWs w = carve(d_ws, cap);
    RG_TRY(flags_pass(t, d_u, p, 1, w.flags, s));
    const int64_t coarse_end = t->level_begin[t->lmin + 1];
    // places of the new octs, and the new level ranges: the octs of level l + 1
    // are the children of the old octs of level l
    const unsigned blocks = static_cast<unsigned>(item_blocks(n));
    Marks old;
    old.n = RG_MAX_LEVEL + 2;
    for (int l = 0; l < old.n; ++l) old.at[l] = l <= t->lmin ? 0 : (l <= t->lmax ? t->level_begin[l] : n);
    k_refine_count<<<blocks, kItems, 0, s>>>(w.flags, t->d_father_cell, n, coarse_end, w.cnt);
    k_scan_blocks<<<1, kItems, 0, s>>>(w.cnt, blocks, w.total);
    k_refine_offsets<<<blocks, kItems, 0, s>>>(w.flags, t->d_father_cell, n, coarse_end, w.cnt, w.total, old, w.off,
                                               w.bound);
    RG_TRY(launch_status("refine offsets"));
    EmitArgs a;
    a.flags = w.flags;
    a.son = t->d_son_mask;
    a.off = w.off;
    a.father = t->d_father_cell;
    a.ijkl = t->d_ijkl;
    a.keys = t->d_keys;
    a.n = n;
    a.coarse_end = coarse_end;
    a.cap = cap;
    a.src = w.src;
    a.new_ijkl = w.new_ijkl;
    a.new_keys = t->d_keys_scratch;
    k_refine_emit<<<grid_for(n, 256), 256, 0, s>>>(a);
    RG_TRY(launch_status("refine emit"));
    int64_t h[RG_MAX_LEVEL + 2];
    if (hipMemcpyAsync(h, w.bound, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return fail(RG_EHIP, "refine count readback");
    const int64_t m = coarse_end + h[RG_MAX_LEVEL + 1];
    if (m > cap)
        return fail(RG_EFULL, "refined tree needs %lld octs, capacity %lld", static_cast<long long>(m),
                    static_cast<long long>(cap));
    Marks lb;
    lb.n = RG_MAX_LEVEL + 2;
    for (int l = 0; l < lb.n; ++l) lb.at[l] = l <= t->lmin ? 0 : coarse_end + h[l - 1];
    const bool wide = aligned(d_u, 16) && aligned(d_u_new, 16) && aligned(t->d_ijkl, 16);
    if (wide)
        k_refine_gather<2><<<grid_for(20 * m, 256), 256, 0, s>>>(w.new_ijkl, t->d_keys_scratch, w.src, d_u, n, m, t->d_ijkl,
                                                                t->d_keys, d_u_new);
    else
        k_refine_gather<1><<<grid_for(40 * m, 256), 256, 0, s>>>(w.new_ijkl, t->d_keys_scratch, w.src, d_u, n, m, t->d_ijkl,
                                                                t->d_keys, d_u_new);
    RG_TRY(launch_status("refine gather"));
    k_refine_levels<<<1, 64, 0, s>>>(t->d_level_begin, lb);
    RG_TRY(launch_status("refine levels"));
    int lmax = t->lmin;
    for (int l = t->lmin; l <= RG_MAX_LEVEL; ++l)
        if (lb.at[l + 1] > lb.at[l]) lmax = l;
    for (int l = 0; l < RG_MAX_LEVEL + 2; ++l) t->level_begin[l] = lb.at[l];
    t->n_oct = m;
    t->lmax = lmax;
    t->sched = nullptr;
    RG_TRY(rg_hash_build(t->d_keys, m, t->d_hash_ws, t->hash_ws_bytes, stream));
    // neighbour lists brick by brick: the complete bricks follow from the
    // keys; the lists' lengths stay on the device, the grids hold as many as
    // there could be.  A complete level of at least 8^3 octs is all bricks.
    int64_t rest = m;
    for (int l = 4; l <= 10; ++l)
        if (lb.at[l + 1] - lb.at[l] == int64_t(1) << (3 * (l - 1))) rest -= lb.at[l + 1] - lb.at[l];
    const size_t core = core_bytes(cap);
    const int32_t *lst = nullptr;
    const uint32_t *d_count = nullptr;
    RG_TRY(nbr_lists_device(t->d_keys, m, t->level_begin, t->lmin, t->lmax, static_cast<char *>(d_ws) + core,
                            ws_bytes - core, &lst, &d_count, s));
    return neighbours_scheduled(t->d_hash_ws, t->d_keys, m, t->lmin, t->lmax, t->level_begin[t->lmax], t->bc, lst,
                                m / 512, lst, rest, t->d_nbr27, t->d_father_cell, t->d_son_mask, s, d_count);
}

}  // extern "C"
