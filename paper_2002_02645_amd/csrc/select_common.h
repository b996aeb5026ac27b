// Device helpers shared by the selection kernels: order-preserving float bits, a bitonic sort
// in LDS, rank counting, sorts within a wave.
#pragma once
#include "freeze_internal.h"

namespace fz {

// fp32 -> unsigned with the same order (so that (key, index) packs into one u64)
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered_bits(uint32_t u)
{
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// What a block of eight entries leaves beside its smallest key (block-minima route), in 16 bits: the place of
// the entry that has it (lowest three bits) and the lead of that key over the block's second smallest, halved, cut off to a
// float of eight exponent and four mantissa bits: never more than the lead is.  Equal keys: no lead.
__device__ __forceinline__ uint32_t block_next(float half_lead, uint32_t at) { return (__float_as_uint(half_lead) >> 16 & 0xfff8u) | at; }
// A lower bound of the keys of a block's other entries from its smallest key.  (The lead is the rounded difference of two
// sums, and twice it is added with another rounding: an ulp of either.)  No number: no bound.
__device__ __forceinline__ float block_others(float key, uint32_t next)
{
    const float lead = 2.f * __uint_as_float((next & 0xfff8u) << 16);
    return key + lead - 2.4e-7f * (__builtin_fabsf(key) + lead);
}

constexpr int kThrThreads = 1024;
constexpr int kThrGroups = 256;
constexpr int kThrList = 8192;    // capacity of the gathered list; callers check V * R <= kThrList

__device__ inline void bitonic_sort_lds(uint64_t *a, int n_pow2, int tid, int nthreads)
{
    for (int size = 2; size <= n_pow2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < (n_pow2 >> 1); i += nthreads) {
                const int lo = ((i & ~(stride - 1)) << 1) | (i & (stride - 1));   // stride is a power of two
                const int hi = lo + stride;
                const bool up = ((lo & size) == 0);
                const uint64_t x = a[lo], y = a[hi];
                if ((x > y) == up) {
                    a[lo] = y;
                    a[hi] = x;
                }
            }
            __syncthreads();
        }
    }
}

// The element of a[0..n) with exactly `rank` smaller elements (all distinct), n <= blockDim.x.
__device__ __forceinline__ void select_by_rank_counting(const uint64_t *a, int n, int rank, int tid, uint64_t *out)
{
    if (tid < n) {
        const uint64_t mine = a[tid];
        int c = 0;
        for (int j = 0; j < n; ++j) c += (a[j] < mine);
        if (c == rank) *out = mine;
    }
}

// Ascending sort of one value per lane across the 64 lanes of a wave (bitonic network on
// register shuffles: no LDS, no barrier).
__device__ __forceinline__ uint64_t wave_sort64(uint64_t x, int lane)
{
#pragma unroll
    for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, stride, 64);
            const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), stride, 64);
            const uint64_t y = ((uint64_t)hi << 32) | lo;
            const bool up = (lane & size) == 0 || size == 64;
            const bool lower = (lane & stride) == 0;
            x = ((x < y) == (lower == up)) ? x : y;   // keep the smaller where lower == up, else the larger
        }
    }
    return x;
}

// The same for 32-bit values.
__device__ __forceinline__ uint32_t wave_sort32(uint32_t x, int lane)
{
#pragma unroll
    for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const uint32_t y = (uint32_t)__shfl_xor((int)x, stride, 64);
            const bool up = (lane & size) == 0 || size == 64;
            const bool lower = (lane & stride) == 0;
            x = ((x < y) == (lower == up)) ? x : y;
        }
    }
    return x;
}

// The `keep` smallest of a[0..cnt), sorted ascending, by the whole workgroup (nthreads a multiple
// of 64): rounds of wave-local sorts of 64 values that each pass on their `keep` smallest, until
// one wave holds the rest.  Needs keep <= 32 (each round at least halves the count) and a second
// buffer b of the same capacity; returns the buffer whose first min(keep, cnt) entries are the
// result.  Every thread must call it; a and b are LDS.
__device__ inline uint64_t *smallest_sorted(uint64_t *a, uint64_t *b, int cnt, int keep, int tid, int nthreads)
{
    const int lane = tid & 63, wave = tid >> 6, nwaves = nthreads >> 6;
    while (true) {
        const int chunks = (cnt + 63) >> 6;
        for (int c = wave; c < chunks; c += nwaves) {
            const int i = c * 64 + lane;
            const uint64_t x = wave_sort64(i < cnt ? a[i] : kSentinel, lane);
            if (chunks == 1) {
                if (lane < 64) b[lane] = x;
            } else if (lane < keep) {
                b[c * keep + lane] = x;
            }
        }
        __syncthreads();
        uint64_t *t = a;
        a = b;
        b = t;
        if (chunks == 1) return a;
        cnt = chunks * keep;   // sentinels may pad the tail: they sort last
    }
}

}  // namespace fz
