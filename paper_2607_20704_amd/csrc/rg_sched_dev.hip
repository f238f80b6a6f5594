// rg_sched_dev.hip -- the kernel schedule built on the device.
//
// Same lists as rg_schedule_build (per level: complete Hilbert-aligned
// 8^3-oct bricks that border no coarse cell, the other octs; every complete
// brick and the other octs for the neighbour build; per level above lmin the
// octs with a coarse cell across a face; per level the complete sibling
// groups outside the bricks and the octs outside bricks and groups), found
// without copying the tree to the host: one pass over the neighbour lists
// notes which octs have a coarse entry and marks their bricks, a second pass
// evaluates the seven membership tests per oct, and the lists are written in
// key order (rg_compact.hpp).  The host reads back only the per-level list
// lengths.  A tree that changes every step (refinement) keeps its brick kernel
// this way.
#include "rg_compact.hpp"
#include "rg_internal.hpp"

namespace rg {
namespace {

// bricks, per-oct, all complete bricks, octs outside them, border octs,
// sibling groups, octs outside bricks and groups
constexpr int kLists = 7;
constexpr int64_t kBrick = 512;      // octs per brick
constexpr int64_t kGroup = 8;        // octs per sibling group
constexpr int kLB = RG_MAX_LEVEL + 2;

struct SchedArgs {
    const uint64_t *keys;
    const int32_t *nbr27;
    int64_t n;
    int64_t begin[kLB];
    int lmin;
};

__device__ __forceinline__ int level_of(const SchedArgs &a, int64_t o)
{
    int l = a.lmin;
    while (l < RG_MAX_LEVEL && o >= a.begin[l + 1]) ++l;
    return l;
}

// first oct of the complete brick holding o, or -1
__device__ __forceinline__ int64_t brick_first(const SchedArgs &a, int64_t o, int l)
{
    const uint64_t k = a.keys[o];
    const int64_t r = static_cast<int64_t>(k & uint64_t(kBrick - 1));
    const int64_t f = o - r;
    if (f < a.begin[l] || f + kBrick - 1 >= a.begin[l + 1]) return -1;
    if (a.keys[f] != k - uint64_t(r) || a.keys[f + kBrick - 1] != k - uint64_t(r) + uint64_t(kBrick - 1)) return -1;
    return f;
}

// first oct of the complete sibling group holding o (levels above lmin), or -1
__device__ __forceinline__ int64_t group_first(const SchedArgs &a, int64_t o, int l)
{
    if (l <= a.lmin) return -1;
    const uint64_t k = a.keys[o];
    const int64_t r = static_cast<int64_t>(k & uint64_t(kGroup - 1));
    const int64_t f = o - r;
    if (f < a.begin[l] || f + kGroup - 1 >= a.begin[l + 1]) return -1;
    if (a.keys[f] != k - uint64_t(r) || a.keys[f + kGroup - 1] != k - uint64_t(r) + uint64_t(kGroup - 1)) return -1;
    return f;
}

__device__ __forceinline__ bool coarse_entry(int32_t v) { return v < 0 && v != RG_NBR_OUTSIDE; }

__global__ void k_sched_zero(uint8_t *p, int64_t n)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Bit 0: some list entry of the oct is a coarse cell; bit 1: one across a
// face.  A complete brick with a coarse entry anywhere in its octs' lists is
// marked in bad[(first oct) / 512] (complete bricks start 512 octs apart at
// least).  The workgroup reads its 256 octs' lists as one stretch, entry
// after entry: 27 words per thread, whole lines (an oct per thread read 108
// bytes apart: 90 us for 1.04 M octs).
__global__ __launch_bounds__(256) void k_sched_mark(SchedArgs a, uint8_t *__restrict__ coarse,
                                                    uint8_t *__restrict__ bad)
{
    __shared__ uint32_t s[256];
    const int t = threadIdx.x;
    const int64_t first = int64_t(blockIdx.x) * 256;
    const int64_t left = 27 * (a.n - first);
    s[t] = 0;
    __syncthreads();
    const int32_t *p = a.nbr27 + 27 * first;
    int k = t / 27, e = t - 27 * (t / 27);   // oct and entry, stepped: 256 = 9 * 27 + 13
#pragma unroll 9
    for (int i = 0; i < 27; ++i) {
        const int q = t + 256 * i;
        const int32_t v = q < left ? p[q] : 0;
        if (coarse_entry(v)) {
            const bool face = e == 4 || e == 10 || e == 12 || e == 14 || e == 16 || e == 22;
            atomicOr(&s[k], face ? 3u : 1u);
        }
        k += 9;
        e += 13;
        if (e >= 27) {
            e -= 27;
            ++k;
        }
    }
    __syncthreads();
    const int64_t o = first + t;
    if (o >= a.n) return;
    coarse[o] = static_cast<uint8_t>(s[t]);
    if (s[t]) {
        const int64_t f = brick_first(a, o, level_of(a, o));
        if (f >= 0) bad[f / kBrick] = 1;
    }
}

struct SchedMember {
    SchedArgs a;
    const uint8_t *coarse, *bad;

    __device__ __forceinline__ uint32_t operator()(int64_t o) const
    {
        const int l = level_of(a, o);
        const int64_t f = brick_first(a, o, l);
        const bool complete = f >= 0;
        const bool covered = complete && bad[f / kBrick] == 0;
        const int64_t g = covered ? -1 : group_first(a, o, l);
        const bool border = l > a.lmin && (coarse[o] & 2);
        return (covered && f == o ? 1u : 0u) | (covered ? 0u : 2u) | (complete && f == o ? 4u : 0u) |
               (complete ? 0u : 8u) | (border ? 16u : 0u) | (g >= 0 && g == o ? 32u : 0u) |
               (!covered && g < 0 ? 64u : 0u);
    }
};

// keys only: first octs of complete bricks (list 0) and octs outside complete
// bricks (list 1), for the brick-wise neighbour build
struct NbrMember {
    SchedArgs a;

    __device__ __forceinline__ uint32_t operator()(int64_t o) const
    {
        const int64_t f = brick_first(a, o, level_of(a, o));
        return (f >= 0 && f == o ? 1u : 0u) | (f < 0 ? 2u : 0u);
    }
};

size_t al(size_t b) { return (b + 255) & ~size_t(255); }

SchedArgs sched_args(const uint64_t *keys, const int32_t *nbr27, int64_t n, const int64_t *begin, int lmin, int lmax)
{
    SchedArgs a;
    a.keys = keys;
    a.nbr27 = nbr27;
    a.n = n;
    for (int l = 0; l < kLB; ++l) a.begin[l] = l <= lmax ? begin[l] : n;
    a.lmin = lmin;
    return a;
}

}  // namespace

size_t nbr_lists_ws_bytes(int64_t n)
{
    n = n > 0 ? n : 1;
    return al(n) + al(8 * item_blocks(n)) + al(4 * n + 4 * (n / kBrick) + 4) + 256;
}

// The neighbour-build lists of a tree from its keys and level ranges alone
// (complete bricks, then the other octs, in key order) into the workspace;
// *list points at them, d_count at the two lengths (device).
rg_status nbr_lists_device(const uint64_t *d_keys, int64_t n, const int64_t *h_level_begin, int lmin, int lmax,
                           void *d_ws, size_t ws_bytes, const int32_t **list, const uint32_t **d_count, hipStream_t s)
{
    RG_REQUIRE(ws_bytes >= nbr_lists_ws_bytes(n) && aligned(d_ws, 256), "neighbour-list workspace too small");
    char *p = static_cast<char *>(d_ws);
    uint32_t *total = reinterpret_cast<uint32_t *>(p);
    p += 256;
    uint8_t *bits = reinterpret_cast<uint8_t *>(p);
    p += al(n);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(p);
    p += al(8 * item_blocks(n));
    int32_t *lst = reinterpret_cast<int32_t *>(p);
    const NbrMember m{sched_args(d_keys, nullptr, n, h_level_begin, lmin, lmax)};
    const unsigned blocks = static_cast<unsigned>(item_blocks(n));
    k_members_count<2><<<blocks, kItems, 0, s>>>(n, m, bits, cnt);
    k_scan_blocks<<<2, kItems, 0, s>>>(cnt, blocks, total);
    Marks none;
    none.n = 0;
    k_members_scatter<2><<<blocks, kItems, 0, s>>>(n, bits, cnt, total, n + n / kBrick + 1, lst, none, nullptr);
    RG_TRY(launch_status("neighbour lists"));
    *list = lst;
    *d_count = total;
    return RG_OK;
}

}  // namespace rg

using namespace rg;

extern "C" {

size_t rg_schedule_workspace_bytes(int64_t n_oct)
{
    const int64_t n = n_oct > 0 ? n_oct : 1;
    return 2 * al(n) + al(n / kBrick + 1) + al(4 * kLists * item_blocks(n)) + al(8 * kLists * kLB) + 512;
}

rg_status rg_schedule_build_device(const rg_tree *t, int32_t *d_list, int64_t capacity, void *d_ws, size_t ws_bytes,
                                   rg_schedule *out, void *stream)
{
    RG_REQUIRE(t && d_list && out && d_ws, "null pointer");
    RG_REQUIRE(t->n_oct > 0 && t->n_oct <= (int64_t(1) << 28) && capacity >= 4 * t->n_oct,
               "list capacity below 4 n_oct");
    RG_REQUIRE(t->lmin >= 1 && t->lmax >= t->lmin && t->lmax <= RG_MAX_LEVEL, "bad levels");
    RG_REQUIRE(t->level_begin[t->lmin] == 0 && t->level_begin[t->lmax + 1] == t->n_oct, "bad level ranges");
    RG_REQUIRE(t->d_keys && t->d_nbr27, "tree without keys or neighbour lists");
    RG_REQUIRE(ws_bytes >= rg_schedule_workspace_bytes(t->n_oct) && aligned(d_ws, 256), "workspace too small");
    const int64_t n = t->n_oct;
    hipStream_t s = as_stream(stream);
    char *p = static_cast<char *>(d_ws);
    uint32_t *lengths = reinterpret_cast<uint32_t *>(p);
    p += 256;
    uint8_t *coarse = reinterpret_cast<uint8_t *>(p);
    p += al(n);
    uint8_t *bits = reinterpret_cast<uint8_t *>(p);
    p += al(n);
    uint8_t *bad = reinterpret_cast<uint8_t *>(p);
    p += al(n / kBrick + 1);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(p);
    p += al(4 * kLists * item_blocks(n));
    int64_t *bounds = reinterpret_cast<int64_t *>(p);

    const SchedArgs a = sched_args(t->d_keys, t->d_nbr27, n, t->level_begin, t->lmin, t->lmax);
    k_sched_zero<<<grid_for(n / kBrick + 1, 256), 256, 0, s>>>(bad, n / kBrick + 1);
    k_sched_mark<<<grid_for(n, 256), 256, 0, s>>>(a, coarse, bad);
    RG_TRY(launch_status("schedule bricks"));
    const SchedMember m{a, coarse, bad};
    const unsigned blocks = static_cast<unsigned>(item_blocks(n));
    k_members_count<kLists><<<blocks, kItems, 0, s>>>(n, m, bits, cnt);
    k_scan_blocks<<<kLists, kItems, 0, s>>>(cnt, blocks, lengths);
    Marks marks;
    marks.n = kLB;
    for (int l = 0; l < kLB; ++l) marks.at[l] = a.begin[l] < n ? a.begin[l] : n;
    k_members_scatter<kLists><<<blocks, kItems, 0, s>>>(n, bits, cnt, lengths, capacity, d_list, marks, bounds);
    RG_TRY(launch_status("schedule lists"));
    int64_t h[kLists * kLB];
    if (hipMemcpyAsync(h, bounds, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return fail(RG_EHIP, "schedule readback");
    auto at = [&](int k, int l) { return h[k * kLB + l]; };
    struct {
        int64_t base[kLists];
    } b;
    int64_t total = 0;
    for (int k = 0; k < kLists; ++k) {
        b.base[k] = total;
        total += at(k, kLB - 1);
    }
    if (total > capacity) return fail(RG_EINVAL, "schedule exceeds list capacity");
    for (int l = 0; l < kLB; ++l)
        out->brick_begin[l] = out->brick_count[l] = out->rest_begin[l] = out->rest_count[l] = out->border_begin[l] =
            out->border_count[l] = out->group_begin[l] = out->group_count[l] = out->single_begin[l] =
                out->single_count[l] = 0;
    for (int l = t->lmin; l <= t->lmax; ++l) {
        out->brick_begin[l] = b.base[0] + at(0, l);
        out->brick_count[l] = at(0, l + 1) - at(0, l);
        out->rest_begin[l] = b.base[1] + at(1, l);
        out->rest_count[l] = at(1, l + 1) - at(1, l);
        if (l > t->lmin) {
            out->border_begin[l] = b.base[4] + at(4, l);
            out->border_count[l] = at(4, l + 1) - at(4, l);
        }
        out->group_begin[l] = b.base[5] + at(5, l);
        out->group_count[l] = at(5, l + 1) - at(5, l);
        out->single_begin[l] = b.base[6] + at(6, l);
        out->single_count[l] = at(6, l + 1) - at(6, l);
    }
    out->nbr_brick_begin = b.base[2];
    out->nbr_brick_count = at(2, kLB - 1);
    out->nbr_rest_begin = b.base[3];
    out->nbr_rest_count = at(3, kLB - 1);
    out->d_list = d_list;
    return RG_OK;
}

}  // extern "C"
