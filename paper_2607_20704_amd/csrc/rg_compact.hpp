// rg_compact.hpp -- lists of an array's members in order, without a library
// scan.
//
// Three launches for any number of lists: per block of 1024 items the members
// of every list are counted (k_members_count, or a count kernel of the
// caller's own), one workgroup per list turns its block counts into offsets
// (k_scan_blocks), and every item finds its place from its block's offset and
// the ballots of its wave (k_members_scatter).  A device-wide scan per list
// cost two launches and two passes over a 32-bit flag and a 32-bit position
// per item and list; the items' membership is one byte here.
#pragma once

#include "rg_internal.hpp"

namespace rg {
namespace {

constexpr int kItems = 1024;   // items and threads of a block

inline int64_t item_blocks(int64_t n) { return (n + kItems - 1) / kItems; }

// exclusive prefix of v over the workgroup's kItems threads and the total;
// s: kItems / 64 words of LDS, free again after the call
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t *s, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) s[wave] = x;
    __syncthreads();
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kItems / 64; ++w) {
        const uint32_t t = s[w];
        before += w < wave ? t : 0u;
        sum += t;
    }
    __syncthreads();
    total = sum;
    return before + x - v;
}

// workgroup k: the block counts cnt[k * nblk ..) into exclusive offsets, in
// place, and their total into total[k]
__global__ __launch_bounds__(kItems) void k_scan_blocks(uint32_t *__restrict__ cnt, int64_t nblk,
                                                        uint32_t *__restrict__ total)
{
    __shared__ uint32_t s[kItems / 64];
    uint32_t *row = cnt + blockIdx.x * nblk;
    uint32_t carry = 0;
    for (int64_t b = 0; b < nblk; b += kItems) {
        const int64_t i = b + threadIdx.x;
        const uint32_t v = i < nblk ? row[i] : 0u;
        uint32_t sum;
        const uint32_t p = block_prefix(v, s, sum);
        if (i < nblk) row[i] = carry + p;
        carry += sum;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// bit k of member(i): item i is in list k; bits[i] and the block counts
template <int K, typename F>
__global__ __launch_bounds__(kItems) void k_members_count(int64_t n, F member, uint8_t *__restrict__ bits,
                                                          uint32_t *__restrict__ cnt)
{
    __shared__ uint32_t c[K];
    if (threadIdx.x < K) c[threadIdx.x] = 0;
    __syncthreads();
    const int64_t i = int64_t(blockIdx.x) * kItems + threadIdx.x;
    const uint32_t m = i < n ? member(i) : 0u;
    if (i < n) bits[i] = static_cast<uint8_t>(m);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = __ballot((m >> k) & 1u);
        if ((threadIdx.x & 63) == 0 && v) atomicAdd(&c[k], static_cast<uint32_t>(__popcll(v)));
    }
    __syncthreads();
    if (threadIdx.x < K) cnt[threadIdx.x * int64_t(gridDim.x) + blockIdx.x] = c[threadIdx.x];
}

// boundaries whose list positions are wanted
struct Marks {
    int n;
    int64_t at[RG_MAX_LEVEL + 2];
};

// list k's items to list[(the lengths of lists 0..k-1) + place], entries past
// `capacity` left out; bound[k * marks.n + j]: list k's members before item
// marks.at[j]
template <int K>
__global__ __launch_bounds__(kItems) void k_members_scatter(int64_t n, const uint8_t *__restrict__ bits,
                                                            const uint32_t *__restrict__ off,
                                                            const uint32_t *__restrict__ total, int64_t capacity,
                                                            int32_t *__restrict__ list, Marks marks,
                                                            int64_t *__restrict__ bound)
{
    __shared__ uint32_t c[K][kItems / 64];
    __shared__ uint64_t in[K][kItems / 64];   // members by wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = int64_t(blockIdx.x) * kItems + threadIdx.x;
    const uint32_t m = i < n ? bits[i] : 0u;
    uint32_t rank[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint64_t v = __ballot((m >> k) & 1u);
        rank[k] = static_cast<uint32_t>(__popcll(v & ((uint64_t(1) << lane) - 1)));
        if (lane == 0) {
            c[k][wave] = static_cast<uint32_t>(__popcll(v));
            in[k][wave] = v;
        }
    }
    __syncthreads();
    // counts of the waves into offsets, one thread per list and wave
    static_assert(K * (kItems / 64) <= kItems, "a thread per list and wave");
    uint32_t before = 0;
    const int ck = threadIdx.x / (kItems / 64), cw = threadIdx.x % (kItems / 64);
    if (ck < K) {
        before = off[ck * int64_t(gridDim.x) + blockIdx.x];
        for (int w = 0; w < cw; ++w) before += c[ck][w];
    }
    __syncthreads();
    if (ck < K) c[ck][cw] = before;
    __syncthreads();
    // one thread per list and boundary (with every thread looking for
    // boundaries at its item 7 lists of 1.04 M items took 43 us instead of 9,
    // most of it in the few blocks that hold one)
    for (int t = threadIdx.x; t < K * marks.n; t += kItems) {
        const int k = t / marks.n;
        const int64_t at = marks.at[t - k * marks.n], q = at - int64_t(blockIdx.x) * kItems;
        if (at >= n) {
            if (blockIdx.x == 0) bound[t] = total[k];
        } else if (q >= 0 && q < kItems) {
            bound[t] = c[k][q >> 6] + __popcll(in[k][q >> 6] & ((uint64_t(1) << (q & 63)) - 1));
        }
    }
    int64_t base = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t pos = c[k][wave] + rank[k];
        if (((m >> k) & 1u) && base + pos < capacity) list[base + pos] = static_cast<int32_t>(i);
        base += total[k];
    }
}

}  // namespace
}  // namespace rg
