// rg_rekey.hip -- keys of a tree's octs in key order.
//
// Paper Sec. 2.2: every step encodes the octs' keys and sorts them by level
// and, inside a level, along the Hilbert curve.  A tree's octs are stored in
// that order (rg.h), so the sort of a step finds nothing to move unless the
// caller changed the coordinates.  The encode therefore writes the keys and
// the identity permutation where the sorted ones go and notes whether any two
// neighbours are out of order; the passes of the sort that follow end at once
// if none are.  A library radix sort went through all its passes either way:
// a step of 0.07 M octs on three levels, with its lists rebuilt, took 203 us
// with it and takes 163 like this; encode, sort and level ranges of 0.26 M
// octs took 94 us and take 28, of 2.1 M 150 and 35, of 16.8 M 843 and 168.
//
// The sort itself (least significant digit first, 8 bits a pass, stable) is
// two launches a pass: digit counts of every tile, then a scatter in which
// every workgroup adds up the counts of the tiles before its own.  With the
// octs in random order the same three calls take 75 us (library: 110), 177
// (141) and 1104 (811).
#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kSortT = 256;        // threads
constexpr int kDigits = 256;       // one per thread
constexpr int kWaves = kSortT / 64;
constexpr int kMaxTiles = 512;     // counts that a scatter adds up per digit

struct SortArgs {
    uint32_t *unsorted;       // some neighbouring keys are out of order
    uint32_t *cnt;            // [tile][digit]
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

// Thread 0 of a workgroup holds the key before the workgroup's own 255.
__global__ __launch_bounds__(256) void k_rekey(const int32_t *__restrict__ ijkl, int64_t n, uint64_t mask,
                                               uint64_t *__restrict__ keys, uint64_t *__restrict__ out,
                                               int32_t *__restrict__ perm, uint32_t *unsorted)
{
    __shared__ uint64_t s[256];
    const int t = threadIdx.x;
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
__device__ __forceinline__ uint64_t same_digit(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool one = (d >> b) & 1u;
        const uint64_t v = __ballot(one);
        m &= one ? v : ~v;
    }
    return m;
}

// exclusive prefix of v over the workgroup; s: kSortT words of LDS
__device__ __forceinline__ uint32_t prefix_of(uint32_t v, uint32_t *s)
{
    const int t = threadIdx.x;
    s[t] = v;
    __syncthreads();
    for (int off = 1; off < kSortT; off <<= 1) {
        const uint32_t x = t >= off ? s[t - off] : 0u;
        __syncthreads();
        s[t] += x;
        __syncthreads();
    }
    const uint32_t r = s[t] - v;
    __syncthreads();
    return r;
}

// Digits of ROUNDS * kSortT keys: wave w holds the keys [w, w + 1) * 64 ROUNDS
// of the part, 64 a round.  hist[w][d]: the wave's keys with digit d; mate[q]:
// lanes of round q with the same digit, before this one and (above 8 bits) in
// all.
template <int ROUNDS>
__device__ __forceinline__ void part_digits(const SortArgs &a, int64_t first, uint64_t *key, uint32_t *mate,
                                            uint32_t (*hist)[kDigits])
{
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) key[q] = first + 64 * q < a.n ? a.src[first + 64 * q] : 0;
    for (int w = 0; w < kWaves; ++w) hist[w][t] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ROUNDS; ++q) {
        const bool valid = first + 64 * q < a.n;
        const uint32_t d = static_cast<uint32_t>(key[q] >> a.shift) & a.dmask;
        const uint64_t m = same_digit(d, valid);
        const uint32_t rank = static_cast<uint32_t>(__popcll(m & ((uint64_t(1) << lane) - 1)));
        const uint32_t all = static_cast<uint32_t>(__popcll(m));
        mate[q] = rank | all << 8;
        if (valid && rank == 0) hist[wave][d] += all;
    }
    __syncthreads();
}

template <int ROUNDS> __device__ __forceinline__ int64_t part_first(const SortArgs &a, int part)
{
    const int64_t p = int64_t(blockIdx.x) * a.parts + part;
    return (p * kWaves + (threadIdx.x >> 6)) * (64 * ROUNDS) + (threadIdx.x & 63);
}

template <int ROUNDS> __global__ __launch_bounds__(kSortT) void k_rekey_count(SortArgs a)
{
    if (*a.unsorted == 0) return;
    __shared__ uint32_t hist[kWaves][kDigits];
    const int t = threadIdx.x;
    uint32_t v = 0;
    for (int part = 0; part < a.parts; ++part) {
        uint64_t key[ROUNDS];
        uint32_t mate[ROUNDS];
        part_digits<ROUNDS>(a, part_first<ROUNDS>(a, part), key, mate, hist);
        for (int w = 0; w < kWaves; ++w) v += hist[w][t];
        __syncthreads();
    }
    a.cnt[int64_t(blockIdx.x) * kDigits + t] = v;
}

template <int ROUNDS> __global__ __launch_bounds__(kSortT) void k_rekey_scatter(SortArgs a)
{
    if (*a.unsorted == 0) return;
    __shared__ uint32_t hist[kWaves][kDigits];
    __shared__ uint32_t scan[kDigits], to[kDigits];
    __shared__ uint64_t skey[ROUNDS * kSortT];
    __shared__ int32_t sval[ROUNDS * kSortT];
    __shared__ uint32_t keys_here;
    const int t = threadIdx.x, wave = t >> 6;
    // per digit: all tiles' counts, and those of the tiles before this one
    uint32_t total = 0, start = 0;
#pragma unroll 8
    for (uint32_t i = 0; i < a.tiles; ++i) {
        const uint32_t v = a.cnt[int64_t(i) * kDigits + t];
        total += v;
        start += i < blockIdx.x ? v : 0u;
    }
    start += prefix_of(total, scan);
    for (int part = 0; part < a.parts; ++part) {
        const int64_t first = part_first<ROUNDS>(a, part);
        uint64_t key[ROUNDS];
        uint32_t mate[ROUNDS];
        part_digits<ROUNDS>(a, first, key, mate, hist);
        // in LDS in digit order first, so that a digit's keys leave together
        // (2.1 M keys in random order: 235 us straight from registers, 177 so)
        uint32_t mine = 0;
        for (int w = 0; w < kWaves; ++w) mine += hist[w][t];
        uint32_t local = prefix_of(mine, scan);
        to[t] = start - local;   // may wrap; so does the sum below
        start += mine;
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t v = hist[w][t];
            hist[w][t] = local;
            local += v;
        }
        if (t == kDigits - 1) keys_here = local;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int64_t i = first + 64 * q;
            const uint32_t d = static_cast<uint32_t>(key[q] >> a.shift) & a.dmask;
            const uint32_t rank = mate[q] & 255u, at = hist[wave][d] + rank;
            __builtin_amdgcn_wave_barrier();
            if (i < a.n) {
                skey[at] = key[q];
                sval[at] = a.val ? a.val[i] : static_cast<int32_t>(i);
                if (rank == 0) hist[wave][d] += mate[q] >> 8;
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        for (uint32_t i = t; i < keys_here; i += kSortT) {
            const uint64_t k = skey[i];
            const uint32_t at = to[static_cast<uint32_t>(k >> a.shift) & a.dmask] + i;
            a.dst[at] = k;
            a.dval[at] = sval[i];
        }
        __syncthreads();
    }
}

size_t al(size_t b) { return (b + 255) & ~size_t(255); }

// Small tiles spread few keys over more compute units; many keys take large
// ones, and beyond kMaxTiles of these several parts to a tile.
constexpr int kFewRounds = 4, kManyRounds = 16;
constexpr int64_t kFewKeys = int64_t(kFewRounds) * kSortT * kMaxTiles;

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

}  // namespace

size_t rekey_workspace_bytes(int64_t n)
{
    n = n > 0 ? n : 1;
    return 256 + al(4 * size_t(kDigits) * tiles_of(n)) + al(8 * n) + al(4 * n);
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
    RG_REQUIRE(end_bit > 0 && end_bit <= 64, "bad key width");
    char *p = static_cast<char *>(d_ws);
    SortArgs a;
    a.unsorted = reinterpret_cast<uint32_t *>(p);
    p += 256;
    a.tiles = tiles_of(n);
    a.parts = parts_of(n);
    a.cnt = reinterpret_cast<uint32_t *>(p);
    p += al(4 * size_t(kDigits) * a.tiles);
    uint64_t *tmp = reinterpret_cast<uint64_t *>(p);
    p += al(8 * n);
    int32_t *tmp_perm = reinterpret_cast<int32_t *>(p);
    a.n = n;
    const uint64_t mask = end_bit == 64 ? ~uint64_t(0) : (uint64_t(1) << end_bit) - 1;
    k_rekey_begin<<<1, 1, 0, s>>>(a.unsorted);
    k_rekey<<<static_cast<unsigned>((n + 254) / 255), 256, 0, s>>>(d_ijkl, n, mask, d_keys, d_sorted, d_perm,
                                                                   a.unsorted);
    RG_TRY(launch_status("rekey"));
    a.src = d_keys;
    a.val = nullptr;
    const int passes = (end_bit + 7) / 8;
    for (int k = 0; k < passes; ++k) {
        // the last pass ends in d_sorted, the others alternate
        const bool to_out = ((passes - 1 - k) & 1) == 0;
        a.dst = to_out ? d_sorted : tmp;
        a.dval = to_out ? d_perm : tmp_perm;
        a.shift = 8 * k;
        const int bits = end_bit - a.shift < 8 ? end_bit - a.shift : 8;
        a.dmask = (1u << bits) - 1u;
        if (rounds_of(n) == kFewRounds) {
            k_rekey_count<kFewRounds><<<a.tiles, kSortT, 0, s>>>(a);
            k_rekey_scatter<kFewRounds><<<a.tiles, kSortT, 0, s>>>(a);
        } else {
            k_rekey_count<kManyRounds><<<a.tiles, kSortT, 0, s>>>(a);
            k_rekey_scatter<kManyRounds><<<a.tiles, kSortT, 0, s>>>(a);
        }
        RG_TRY(launch_status("rekey sort"));
        a.src = a.dst;
        a.val = a.dval;
    }
    return RG_OK;
}

}  // namespace rg
