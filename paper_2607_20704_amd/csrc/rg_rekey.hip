// rg_rekey.hip -- keys of a tree's octs in key order.
//
// Paper Sec. 2.2: every step encodes the octs' keys and sorts them by level
// and, inside a level, along the Hilbert curve.  A tree's octs are stored in
// that order (rg.h), so the sort of a step finds nothing to move unless the
// caller changed the coordinates.  The encode therefore writes the keys and
// the identity permutation where the sorted ones go and notes whether any two
// neighbours are out of order; the passes of the sort that follow end at once
// if none are, and sort everything if one pair is.  A library radix sort went
// through all its passes either way.
//
// The sort itself (least significant digit first, 8 or 9 bits a pass, stable)
// is two launches a pass: digit counts of every tile, then a scatter in which
// every workgroup adds up the counts of the tiles before its own.  Those come
// in groups of 64 tiles, added up while they were made: with a sum over up to
// 512 tiles in every workgroup a pass over 2.1 M keys took 47 us, 40 of them in
// that chain of loads (21 us now).  Nine bits a pass where that saves a pass.
//
// Encode, sort and level ranges in us, with the library's sort and like this:
//     octs      bits   in order     one pair swapped   random order
//     0.03 M    18     50    25      52    38            51    38
//     0.26 M    21    101    30     101    58           121    58
//     0.50 M    24    130    32     129    68           157    67
//     2.1 M     24    153    41     154   106           145   104
//     2.1 M     30    190    47     186   126           182   125
//     4.2 M     27    310    59     309   206           299   205
//     16.8 M    27    848   177     847   712           815   715
//     16.8 M    30    827   190     830   763           814   761
#include <algorithm>
#include <utility>

#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kSortT = 256;        // threads
constexpr int kWaves = kSortT / 64;
constexpr int kMaxBits = 9;        // of a digit
constexpr int kMaxPasses = 7;      // 63 bits
constexpr int kGroupTiles = 64;    // tiles whose counts are added up as they are made

struct SortArgs {
    uint32_t *unsorted;       // some neighbouring keys are out of order
    uint32_t *cnt;            // [tile][digit]
    uint32_t *sum;            // [group of kGroupTiles tiles][digit], zero before the pass
    uint32_t *next_sum;       // the next pass's, cleared by this one's scatter
    uint32_t nsum;            // words of either
    const uint64_t *src;
    const int32_t *val;       // nullptr in the first pass: the index itself
    uint64_t *dst;
    int32_t *dval;
    int64_t n;
    uint32_t tiles;
    int parts;                // of ROUNDS * kSortT keys per tile
    int shift;
    uint32_t dmask;
};

__global__ void k_rekey_begin(uint32_t *unsorted) { *unsorted = 0; }

// Thread 0 of a workgroup holds the key before the workgroup's own 255.  sum:
// the group counts, cleared here for the sort.
__global__ __launch_bounds__(256) void k_rekey(const int32_t *__restrict__ ijkl, int64_t n, uint64_t mask,
                                               uint64_t *__restrict__ keys, uint64_t *__restrict__ out,
                                               int32_t *__restrict__ perm, uint32_t *unsorted,
                                               uint32_t *__restrict__ sum, uint32_t nsum)
{
    __shared__ uint64_t s[256];
    const int t = threadIdx.x;
    for (int64_t i = int64_t(blockIdx.x) * 256 + t; i < nsum; i += int64_t(gridDim.x) * 256) sum[i] = 0;
    const int64_t o = int64_t(blockIdx.x) * 255 + t - 1;
    uint64_t k = 0;
    if (o >= 0 && o < n) {
        const int4 c = reinterpret_cast<const int4 *>(ijkl)[o];
        k = oct_key(c.x, c.y, c.z, c.w);
    }
    s[t] = k;
    __syncthreads();
    if (t == 0 || o >= n) return;
    keys[o] = k;
    out[o] = k;
    perm[o] = static_cast<int32_t>(o);
    if (o > 0 && (s[t - 1] & mask) > (k & mask)) *unsorted = 1;
}

// lanes of the wave with this lane's digit
template <int BITS> __device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool one = (d >> b) & 1u;
        const uint64_t v = __ballot(one);
        m &= one ? v : ~v;
    }
    return m;
}

// v[0..E) of the workgroup's threads, in order, into their exclusive prefix;
// s: kSortT words of LDS
template <int E> __device__ __forceinline__ void prefix_of(uint32_t (&v)[E], uint32_t *s)
{
    const int t = threadIdx.x;
    uint32_t mine = 0;
#pragma unroll
    for (int h = 0; h < E; ++h) mine += v[h];
    s[t] = mine;
    __syncthreads();
    for (int off = 1; off < kSortT; off <<= 1) {
        const uint32_t x = t >= off ? s[t - off] : 0u;
        __syncthreads();
        s[t] += x;
        __syncthreads();
    }
    uint32_t before = s[t] - mine;
#pragma unroll
    for (int h = 0; h < E; ++h) {
        const uint32_t x = v[h];
        v[h] = before;
        before += x;
    }
    __syncthreads();
}

// Tile of a workgroup: each XCD takes a contiguous eighth of the tiles, whose
// stretches of a digit adjoin and so share lines of its L2.  The grid has
// 8 ceil(tiles / 8) workgroups.
__device__ __forceinline__ uint32_t tile_of_block(const SortArgs &a)
{
    return blockIdx.x % 8 * ((a.tiles + 7) / 8) + blockIdx.x / 8;
}

// A part is ROUNDS * kSortT keys: wave w holds the keys [w, w + 1) * 64 ROUNDS
// of it, 64 a round.  The thread's first key:
template <int ROUNDS> __device__ __forceinline__ int64_t part_first(const SortArgs &a, uint32_t tile, int part)
{
    const int64_t p = int64_t(tile) * a.parts + part;
    return (p * kWaves + (threadIdx.x >> 6)) * (64 * ROUNDS) + (threadIdx.x & 63);
}

// keys from there to the end (the thread's round q has one if 64 q is below)
template <int ROUNDS> __device__ __forceinline__ int part_left(const SortArgs &a, int64_t first)
{
    return static_cast<int>(min(max(a.n - first, int64_t(0)), int64_t(64 * ROUNDS)));
}

// Bound by the read of the keys.  A tile's digits, added up in LDS; a round whose lanes all have one digit
// (the high digits of keys nearly in order) is one addition.
template <int BITS, int ROUNDS> __global__ __launch_bounds__(kSortT) void k_rekey_count(SortArgs a)
{
    if (*a.unsorted == 0) return;
    const uint32_t tile = tile_of_block(a);
    if (tile >= a.tiles) return;
    constexpr int D = 1 << BITS;
    __shared__ uint32_t hist[D];
    const int t = threadIdx.x;
    for (int d = t; d < D; d += kSortT) hist[d] = 0;
    __syncthreads();
    for (int part = 0; part < a.parts; ++part) {
        const int64_t first = part_first<ROUNDS>(a, tile, part);
        const int left = part_left<ROUNDS>(a, first);
        const uint64_t *src = a.src + first;
        uint64_t key[ROUNDS];
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) key[q] = 64 * q < left ? src[64 * q] : 0;
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q)
            if (64 * q < left) {
                const uint32_t d = static_cast<uint32_t>(key[q] >> a.shift) & a.dmask;
                const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
                if (__ballot(d != d0) == 0) {
                    const uint64_t m = __ballot(1);
                    if (__ffsll(static_cast<unsigned long long>(m)) - 1 == (t & 63))
                        atomicAdd(&hist[d0], static_cast<uint32_t>(__popcll(m)));
                } else {
                    atomicAdd(&hist[d], 1u);
                }
            }
    }
    __syncthreads();
    for (int d = t; d < D; d += kSortT) {
        const uint32_t v = hist[d];
        a.cnt[tile * D + d] = v;
        if (v) atomicAdd(&a.sum[tile / kGroupTiles * D + d], v);
    }
}

// Bound by memory: 12 bytes read and 12 written per key, the writes a digit's
// stretch of a tile at a time (four or eight keys), which have to meet in the
// L2 to leave as whole lines.  The keys and values read once pass by the
// caches for that (16.8 M keys: 771 us for the whole call without, 715 so),
// and the values are staged where the keys were, so that the registers and not
// the LDS set how many workgroups a compute unit holds (four; with both
// staged, 16 rounds and 54 KB it held two, and a pass over 16.8 M keys took
// 235 us, 180 now).
template <int BITS, int ROUNDS> __global__ __launch_bounds__(kSortT) void k_rekey_scatter(SortArgs a)
{
    if (*a.unsorted == 0) return;
    const uint32_t tile = tile_of_block(a);
    if (tile >= a.tiles) return;
    constexpr int D = 1 << BITS, E = D / kSortT;   // E digits per thread: E t .. E t + E - 1
    static_assert(E >= 1, "a digit per thread at least");
    __shared__ uint32_t hist[kWaves][D];   // the wave's keys with each digit, then where they go
    __shared__ uint32_t scan[kSortT], to[D];
    __shared__ union {
        uint64_t key[ROUNDS * kSortT];
        int32_t val[ROUNDS * kSortT];   // once the keys have left
    } stage;
    __shared__ uint32_t keys_here;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    for (uint32_t i = tile * kSortT + t; i < a.nsum; i += a.tiles * kSortT) a.next_sum[i] = 0;
    // per digit: all tiles' counts, and those of the tiles before this one
    const uint32_t group = tile / kGroupTiles, groups = (a.tiles + kGroupTiles - 1) / kGroupTiles;
    uint32_t total[E] = {}, start[E] = {};
#pragma unroll 8
    for (uint32_t i = 0; i < groups; ++i)
#pragma unroll
        for (int h = 0; h < E; ++h) {
            const uint32_t v = a.sum[i * D + E * t + h];
            total[h] += v;
            start[h] += i < group ? v : 0u;
        }
#pragma unroll 8
    for (uint32_t i = group * kGroupTiles; i < tile; ++i)
#pragma unroll
        for (int h = 0; h < E; ++h) start[h] += a.cnt[i * D + E * t + h];
    prefix_of<E>(total, scan);
#pragma unroll
    for (int h = 0; h < E; ++h) start[h] += total[h];
    for (int part = 0; part < a.parts; ++part) {
        const int64_t first = part_first<ROUNDS>(a, tile, part);
        const int left = part_left<ROUNDS>(a, first);
        uint64_t key[ROUNDS];
        uint32_t mate[ROUNDS], place[ROUNDS];
        int32_t val[ROUNDS];
        const uint64_t *src = a.src + first;
        const int32_t *src_val = a.val + first;
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) key[q] = 64 * q < left ? __builtin_nontemporal_load(src + 64 * q) : 0;
        for (int i = t; i < kWaves * D; i += kSortT) (&hist[0][0])[i] = 0;
        __syncthreads();
        // mate: lanes of the round with the same digit, before this one and
        // (above 8 bits) in all
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const bool valid = 64 * q < left;
            const uint32_t d = static_cast<uint32_t>(key[q] >> a.shift) & a.dmask;
            const uint64_t m = same_digit<BITS>(d, valid);
            const uint32_t rank = static_cast<uint32_t>(__popcll(m & ((uint64_t(1) << lane) - 1)));
            const uint32_t all = static_cast<uint32_t>(__popcll(m));
            mate[q] = rank | all << 8;
            if (valid && rank == 0) hist[wave][d] += all;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q)
            val[q] = !a.val ? static_cast<int32_t>(first) + 64 * q : (64 * q < left ? __builtin_nontemporal_load(src_val + 64 * q) : 0);
        // in LDS in digit order first, so that a digit's keys leave together
        uint32_t local[E];
#pragma unroll
        for (int h = 0; h < E; ++h) {
            local[h] = 0;
            for (int w = 0; w < kWaves; ++w) local[h] += hist[w][E * t + h];
        }
        uint32_t mine[E];
#pragma unroll
        for (int h = 0; h < E; ++h) mine[h] = local[h];
        prefix_of<E>(local, scan);
        const uint32_t end = local[E - 1] + mine[E - 1];
#pragma unroll
        for (int h = 0; h < E; ++h) {
            to[E * t + h] = start[h] - local[h];   // may wrap; so does the sum below
            start[h] += mine[h];
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t v = hist[w][E * t + h];
                hist[w][E * t + h] = local[h];
                local[h] += v;
            }
        }
        if (t == kSortT - 1) keys_here = end;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const uint32_t d = static_cast<uint32_t>(key[q] >> a.shift) & a.dmask;
            const uint32_t rank = mate[q] & 255u, all = mate[q] >> 8;
            mate[q] = hist[wave][d] + rank;   // the key's place in LDS from here on
            __builtin_amdgcn_wave_barrier();
            if (64 * q < left) {
                stage.key[mate[q]] = key[q];
                if (rank == 0) hist[wave][d] += all;
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const uint32_t i = t + kSortT * q;
            if (i < keys_here) {
                const uint64_t k = stage.key[i];
                place[q] = to[static_cast<uint32_t>(k >> a.shift) & a.dmask] + i;
                a.dst[place[q]] = k;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q)
            if (64 * q < left) stage.val[mate[q]] = val[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q)
            if (t + kSortT * q < keys_here) a.dval[place[q]] = stage.val[t + kSortT * q];
        __syncthreads();
    }
}

size_t al(size_t b) { return (b + 255) & ~size_t(255); }

// Small tiles spread few keys over more compute units; many keys take large
// ones, and beyond kMaxTiles of these several parts to a tile.
constexpr int kFewRounds = 4, kManyRounds = 8;
constexpr int64_t kFewKeys = 1 << 19;
constexpr int kMaxTiles = 4096;

int rounds_of(int64_t n) { return n <= kFewKeys ? kFewRounds : kManyRounds; }

int parts_of(int64_t n)
{
    const int64_t part = int64_t(rounds_of(n)) * kSortT;
    return static_cast<int>((n + part * kMaxTiles - 1) / (part * kMaxTiles));
}

uint32_t tiles_of(int64_t n)
{
    const int64_t tile = int64_t(rounds_of(n)) * kSortT * parts_of(n);
    return static_cast<uint32_t>((n + tile - 1) / tile);
}

// Tiles that the workspace has tables for: at least as many as any smaller n
// has, although the tiles become fewer where they become larger.
uint32_t table_tiles(int64_t n)
{
    if (n <= kFewKeys) return tiles_of(n);
    const int64_t one_part = int64_t(kManyRounds) * kSortT * kMaxTiles;
    return n > one_part ? kMaxTiles : std::max(tiles_of(kFewKeys), tiles_of(n));
}

// words of one pass's group counts
uint32_t sums_of(int64_t n) { return (table_tiles(n) + kGroupTiles - 1) / kGroupTiles << kMaxBits; }

template <int BITS> void sort_pass(const SortArgs &a, bool few, hipStream_t s)
{
    const unsigned blocks = 8 * ((a.tiles + 7) / 8);
    if (few) {
        k_rekey_count<BITS, kFewRounds><<<blocks, kSortT, 0, s>>>(a);
        k_rekey_scatter<BITS, kFewRounds><<<blocks, kSortT, 0, s>>>(a);
    } else {
        k_rekey_count<BITS, kManyRounds><<<blocks, kSortT, 0, s>>>(a);
        k_rekey_scatter<BITS, kManyRounds><<<blocks, kSortT, 0, s>>>(a);
    }
}

}  // namespace

size_t rekey_workspace_bytes(int64_t n)
{
    n = n > 0 ? n : 1;
    return 256 + al((size_t(4) << kMaxBits) * table_tiles(n)) + 2 * al(4 * size_t(sums_of(n))) + al(8 * n) + al(4 * n);
}

// Keys of the octs d_ijkl into d_keys, sorted over their low end_bit bits into
// d_sorted with d_perm their places before (stable).
rg_status rekey(const int32_t *d_ijkl, int64_t n, uint64_t *d_keys, uint64_t *d_sorted, int32_t *d_perm, void *d_ws,
                size_t ws_bytes, int end_bit, hipStream_t s)
{
    RG_REQUIRE(n > 0 && n <= INT32_MAX, "n out of range");
    RG_REQUIRE(d_ijkl && d_keys && d_sorted && d_perm && d_ws, "null pointer");
    RG_REQUIRE(aligned(d_ijkl, 16) && aligned(d_keys, 8), "misaligned pointer");
    RG_REQUIRE(d_keys != d_sorted, "in-place sort is not supported");
    RG_REQUIRE(ws_bytes >= rg_sort_workspace_bytes(n), "sort workspace too small");
    RG_REQUIRE(aligned(d_ws, 256), "workspace must be 256-byte aligned");
    RG_REQUIRE(end_bit > 0 && end_bit <= kMaxPasses * kMaxBits, "bad key width");
    const int passes = (end_bit + kMaxBits - 1) / kMaxBits, width = (end_bit + passes - 1) / passes;
    char *p = static_cast<char *>(d_ws);
    SortArgs a;
    a.unsorted = reinterpret_cast<uint32_t *>(p);
    p += 256;
    a.tiles = tiles_of(n);
    a.parts = parts_of(n);
    a.cnt = reinterpret_cast<uint32_t *>(p);
    p += al((size_t(4) << kMaxBits) * table_tiles(n));
    a.nsum = sums_of(n);
    a.sum = reinterpret_cast<uint32_t *>(p);
    p += al(4 * size_t(a.nsum));
    a.next_sum = reinterpret_cast<uint32_t *>(p);
    p += al(4 * size_t(a.nsum));
    uint64_t *tmp = reinterpret_cast<uint64_t *>(p);
    p += al(8 * n);
    int32_t *tmp_perm = reinterpret_cast<int32_t *>(p);
    a.n = n;
    const uint64_t mask = (uint64_t(1) << end_bit) - 1;
    k_rekey_begin<<<1, 1, 0, s>>>(a.unsorted);
    k_rekey<<<static_cast<unsigned>((n + 254) / 255), 256, 0, s>>>(d_ijkl, n, mask, d_keys, d_sorted, d_perm,
                                                                   a.unsorted, a.sum, a.nsum);
    RG_TRY(launch_status("rekey"));
    a.src = d_keys;
    a.val = nullptr;
    for (int k = 0; k < passes; ++k) {
        // the last pass ends in d_sorted, the others alternate
        const bool to_out = ((passes - 1 - k) & 1) == 0;
        a.dst = to_out ? d_sorted : tmp;
        a.dval = to_out ? d_perm : tmp_perm;
        a.shift = width * k;
        const int bits = end_bit - a.shift < width ? end_bit - a.shift : width;
        a.dmask = (1u << bits) - 1u;
        if (width > 8) sort_pass<9>(a, n <= kFewKeys, s);
        else sort_pass<8>(a, n <= kFewKeys, s);
        RG_TRY(launch_status("rekey sort"));
        a.src = a.dst;
        a.val = a.dval;
        std::swap(a.sum, a.next_sum);
    }
    return RG_OK;
}

}  // namespace rg
