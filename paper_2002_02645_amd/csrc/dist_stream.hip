// Distance pass for serving batches (at most 128 queries, any activation length), for up to 1,024 queries on
// small caches, and for projections of up to 512 inputs: every ranking key is written out (or every output), the
// selection is left to keys_finish_kernel.
//
// With 128 queries or fewer the pass is bound by reading the cache once from HBM: a tile of 256
// entries x 32 elements is 16 KiB, 0.6 us of a CU's share of the memory rate, and 128 x 256 x 32
// multiply-adds on it take a third of that.  The 256-query tile of the batched kernel does the
// matrix work for 256 rows whatever the batch, which made a single request as expensive as 256 of
// them (50,000 x 16,384: 381 us for a 231 us stream).  So the query tile here is 16, 32, 64 or 128
// rows, and the kernel is built like the small-batch one: a stream with many bytes in flight.
//
//   - Work: the flattened space (query tile, cache tile, k-step of 32 elements) is cut into equal
//     ranges, one per workgroup, at most two workgroups per CU (one's end of a tile overlaps the other's
//     stream); look-ups take ranges of whole tiles where that is faster (plan_stream).  A tile that lies in one range is finished in place; a tile cut by a range's end
//     leaves its accumulators, BM x 256 fp32 (16 - 128 KiB), in a slot per piece, and
//     stream_fixup_kernel adds the pieces up in a fixed order.
//   - A k-step's stage in LDS is 16 KiB of cache and BM x 64 bytes of queries, both exact copies of
//     the tiled layout, fetched with LDS-direct loads into a ring of NS stages.  The ring runs on
//     across tile boundaries; the kernel counts its own loads and stores (stores are issued through
//     inline asm so that their number is known) and never drains the queue inside its range.
//   - The matrix instruction takes entries as its rows and queries as its columns: a lane then holds
//     four consecutive entries of one query, so keys leave as 16-byte stores straight from the
//     accumulators, and the minimum of a block of 32 entries is an in-lane minimum and two shuffles.
//
// What it takes (whole look-ups, batched kernel -> this one with ranges cut evenly -> with whole tiles):
// 50,000 x 16,384, one query 460 -> 294 -> 264 us (this kernel 257 us = 6.4 TB/s cut, 231 us whole, where a pure read
// reaches 7.1 TB/s; on another card 299 -> 306); 50,000 x 8,192, 32 queries 296 -> 182 -> 153 us (148 us = 5.5 TB/s
// cut, 119 us whole).  Cut: 20,000 x 16,384, 64 / 128 queries 250 -> 179 / 255 -> 213 us.  Short tiles, never cut: 300,000 x
// 512, 64 queries 172 -> 115 us.  At 160 queries a 256-row tile is as fast on a large cache, so 128 is the last size served there.
//
// Paper: Sec. 3 (k nearest neighbours of the layer output), Sec. 5 "Cache lookup performance".
#include "freeze_internal.h"
#include "select_common.h"

#include <algorithm>
#include <cmath>

namespace fz {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

namespace {

constexpr int kEntryBytes = kTileN * kKB * 2;   // 16 KiB: one k-block of one cache tile
constexpr int kNormBytes = 2 * 8 * 256;         // per tile parity and wave, 64 floats

// BM queries per tile; WQ waves share the tile's queries (the other 8 / WQ its entries)
template <int BM_, int WQ_, int NS_>
struct StreamCfg {
    static constexpr int BM = BM_, WQ = WQ_, NS = NS_;
    static constexpr int WE = 8 / WQ;
    static constexpr int EB = kTileN / 16 / WE;      // 16-entry blocks per wave
    static constexpr int QB = BM / 16 / WQ;          // 16-query blocks per wave
    static constexpr int A_BYTES = BM * kKB * 2;
    static constexpr int STAGE = kEntryBytes + A_BYTES;
    static constexpr int NQI = A_BYTES / 1024;       // query loads per stage: one each by waves 0 .. NQI - 1
    static constexpr int LDS_BYTES = NS * STAGE + kNormBytes;
    static constexpr int STORES = EB * QB + (EB / 2) * QB;   // per wave and finished tile: keys, block minima
    static_assert(NQI >= 1 && NQI <= 8 && EB % 2 == 0, "load split, whole blocks of 32 entries");
    static_assert(LDS_BYTES <= 81920, "two workgroups per CU");
    static_assert((NS - 2) * 3 + STORES <= 63, "vmcnt range");
};

struct StreamArgs {
    const uint16_t *q_bf;   // tiled, tiles of BM rows
    const uint16_t *c_bf;   // tiled, tiles of 256 rows
    const float *norm;
    float *keys;            // [m_tiles * BM, n_pad]
    uint64_t *bmin;         // [m_tiles * BM, n_pad / 32]
    float *partial;         // [workgroups, 2] slots of BM x 256 fp32 in fragment order
    const int32_t *count;   // device: live queries, or null (= b)
    int b, n_tiles, nk;     // nk = k-steps per tile
    int64_t len;            // k-steps per workgroup
    int64_t n_pad;
    int once;               // one query tile: the cache is read once and its loads carry the non-temporal hint
    // as a projection: keys [b, ld] = acc + norm[col] (the bias), optionally through ReLU; no block minima,
    // nothing is written past row b or column n
    int projection, relu, n;
    int64_t ld;
};

__device__ __forceinline__ void load4_to_lds(uint64_t sbase, uint32_t voff, uint32_t lds_byte_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase) : "memory", "m0");
}
// Stores whose number the kernel knows (they share the counter of the loads).  The compiler does not know
// them for stores: the no-op keeps the next instruction from overwriting the last of the 16 bytes before
// the store has read it (8-byte stores need none).  Only for values that vector instructions made: nothing
// here waits for a matrix result.
__device__ __forceinline__ void store16(void *p, f32x4 v) { asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" ::"v"(p), "v"(v) : "memory"); }
__device__ __forceinline__ void store8(void *p, u32x2 v) { asm volatile("global_store_dwordx2 %0, %1, off" ::"v"(p), "v"(v) : "memory"); }

__device__ __forceinline__ uint64_t min_u64_xor(uint64_t x, int off)
{
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, off, 64);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), off, 64);
    const uint64_t o = ((uint64_t)hi << 32) | lo;
    return o < x ? o : x;
}

// Keys and block minima of one wave's part of a finished tile.  nrm[cb]: the norms of entries
// 16 cb + 4 (lane >> 4) .. + 3 of the wave's part.  Rows past the batch are written too (the buffers have
// m_tiles * BM rows): the number of stores is the same for every wave.
template <class C>
__device__ __forceinline__ void emit_tile(const f32x4 (&acc)[C::EB][C::QB], const f32x4 (&nrm)[C::EB], const StreamArgs &p, int mt,
                                          int nt, int we, int wq, int lane)
{
    const int e0 = nt * kTileN + we * C::EB * 16 + (lane >> 4) * 4;   // first of the lane's entries in block 0
    if (p.projection) {   // uniform
        const bool vec = (p.ld % 4) == 0;   // rows of whole 16-byte pieces (the buffer is 16-byte aligned)
        const int nq = p.count ? *p.count : p.b;
#pragma unroll
        for (int qb = 0; qb < C::QB; ++qb) {
            const int64_t row = (int64_t)mt * C::BM + (wq * C::QB + qb) * 16 + (lane & 15);
            if (row < nq) {
#pragma unroll
                for (int cb = 0; cb < C::EB; ++cb) {
                    const int col = e0 + cb * 16;
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[cb][qb][e] + nrm[cb][e];
                        if (p.relu) v[e] = __builtin_fmaxf(v[e], 0.f);
                    }
                    float *dst = p.keys + row * p.ld + col;
                    if (vec && col + 4 <= p.n) {
                        *reinterpret_cast<f32x4 *>(dst) = v;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (col + e < p.n) dst[e] = v[e];
                    }
                }
            }
        }
        return;
    }
#pragma unroll
    for (int qb = 0; qb < C::QB; ++qb) {
        const int64_t row = (int64_t)mt * C::BM + (wq * C::QB + qb) * 16 + (lane & 15);
        float *krow = p.keys + row * p.n_pad + e0;
        uint64_t mn = kSentinel;
#pragma unroll
        for (int cb = 0; cb < C::EB; ++cb) {
            f32x4 key;
#pragma unroll
            for (int e = 0; e < 4; ++e) key[e] = __builtin_fmaf(-2.f, acc[cb][qb][e], nrm[cb][e]);
            store16(krow + cb * 16, key);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint64_t pr = ((uint64_t)ordered_bits(key[e]) << 32) | (uint32_t)(e0 + cb * 16 + e);
                mn = pr < mn ? pr : mn;
            }
            if (cb & 1) {
                mn = min_u64_xor(mn, 16);
                mn = min_u64_xor(mn, 32);
                // (the four lanes of a query store the same value)
                store8(p.bmin + row * (p.n_pad / 32) + nt * (kTileN / 32) + we * (C::EB / 2) + (cb >> 1),
                       u32x2{(uint32_t)mn, (uint32_t)(mn >> 32)});
                mn = kSentinel;
            }
            __builtin_amdgcn_sched_barrier(0);   // one block at a time: keeps the registers within two workgroups per CU
        }
    }
}

template <class C>
__global__ __launch_bounds__(512, 4) void dist_stream_kernel(StreamArgs p)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[C::LDS_BYTES];
    constexpr int NS = C::NS, NORMS = NS * C::STAGE;
    const bf16x8 *smem16 = reinterpret_cast<const bf16x8 *>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int we = w % C::WE, wq = w / C::WE;
    const int nq = p.count ? *p.count : p.b;
    const int live_mt = (nq + C::BM - 1) / C::BM;
    const int64_t total = (int64_t)live_mt * p.n_tiles * p.nk;
    const int64_t g0 = (int64_t)blockIdx.x * p.len;
    if (g0 >= total) return;   // uniform
    const int steps = (int)(g0 + p.len < total ? p.len : total - g0);
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
    const bool loads_q = w < C::NQI;   // this wave fetches 1 KiB of queries per stage

    // cursor of the loads: k-step kb of tile (mt, nt); it stops at the range's last step, which the
    // refills past the end repeat (never read), so that the number of outstanding loads stays uniform
    const int tile0 = (int)(g0 / p.nk);
    int i_kb = (int)(g0 - (int64_t)tile0 * p.nk), i_nt = tile0 % p.n_tiles, i_mt = tile0 / p.n_tiles;
    int i_left = steps;
    const uint64_t cbase = (uint64_t)(uintptr_t)p.c_bf, qbase = (uint64_t)(uintptr_t)p.q_bf;
    const uint32_t lane_off = w * 1024 + lane * 16;
    auto issue = [&](int slot) {
        const uint64_t src = uniform_u64(cbase + ((uint64_t)i_nt * p.nk + i_kb) * kEntryBytes);
        const uint32_t dst = smem_base + slot * C::STAGE + w * 1024;
        if (p.once) {   // uniform
            load16_global_to_lds_nt(src, lane_off, dst);
            load16_global_to_lds_nt(src + 8192, lane_off, dst + 8192);
        } else {
            load16_global_to_lds(src, lane_off, dst);
            load16_global_to_lds(src + 8192, lane_off, dst + 8192);
        }
        if (loads_q) {
            const uint64_t qsrc = uniform_u64(qbase + ((uint64_t)i_mt * p.nk + i_kb) * C::A_BYTES);
            load16_global_to_lds(qsrc, lane_off, dst + kEntryBytes);
        }
        if (i_left > 1) {
            --i_left;
            if (++i_kb == p.nk) {
                i_kb = 0;
                if (++i_nt == p.n_tiles) {
                    i_nt = 0;
                    ++i_mt;
                }
            }
        }
    };
    // norms of the wave's entries of cache tile nt -> buffer `par`
    auto issue_norms = [&](int nt, int par) {
        load4_to_lds(uniform_u64((uint64_t)(uintptr_t)(p.norm + (size_t)nt * kTileN + we * C::EB * 16)), (lane & (C::EB * 16 - 1)) * 4,
                     smem_base + NORMS + (par * 8 + w) * 256);
    };

    int kb = i_kb, nt = i_nt, mt = i_mt, par = 0;
    issue_norms(nt, 0);
#pragma unroll
    for (int ps = 0; ps < NS - 1; ++ps) issue(ps);

    // fragment addresses in 16-byte units relative to a stage (lane l: row l & 15 of the block, chunk l >> 4;
    // rows 16 apart share their swizzle)
    const int rdE = (we * C::EB * 16 + (lane & 15)) * 4 + ((lane >> 4) ^ tiled_chunk_swizzle(lane & 15));
    const int rdQ = kEntryBytes / 16 + (wq * C::QB * 16 + (lane & 15)) * 4 + ((lane >> 4) ^ tiled_chunk_swizzle(lane & 15));

    f32x4 acc[C::EB][C::QB];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < C::EB; ++i)
#pragma unroll
            for (int j = 0; j < C::QB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    int slot = 0;
    int seg_kb = kb;          // where the current segment of the tile starts
    int since = NS;           // steps since the last stores
    int seg_steps = 0;
    for (int gs = 0; gs < steps; ++gs) {
        // The stage of this step must have landed: the wave's own loads first, then everyone's (barrier).
        // Younger than them are the loads of NS - 2 stages, and the stores of a tile finished within the
        // last NS - 1 steps.  The barrier also says that every wave has read the stage of the step before,
        // which is refilled next.
        const bool st = since < NS;
        if (loads_q) {
            if (st) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * 3 + C::STORES) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * 3) : "memory");
        } else {
            if (st) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * 2 + C::STORES) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NS - 2) * 2) : "memory");
        }
        ++since;
        ++seg_steps;
        // the next tile's norms, older than every stage that will be in flight when they are read
        if (seg_steps == 1 && gs + (p.nk - kb) < steps) issue_norms(nt + 1 == p.n_tiles ? 0 : nt + 1, par ^ 1);
        issue(slot == 0 ? NS - 1 : slot - 1);

        bf16x8 ef[C::EB], qf[C::QB];
        const int base = slot * (C::STAGE / 16);
#pragma unroll
        for (int i = 0; i < C::EB; ++i) ef[i] = smem16[base + rdE + i * 64];
#pragma unroll
        for (int j = 0; j < C::QB; ++j) qf[j] = smem16[base + rdQ + j * 64];
#pragma unroll
        for (int i = 0; i < C::EB; ++i)
#pragma unroll
            for (int j = 0; j < C::QB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ef[i], qf[j], acc[i][j], 0, 0, 0);
        slot = slot + 1 == NS ? 0 : slot + 1;
        ++kb;
        if (kb < p.nk && gs + 1 < steps) continue;

        // ---- the tile, or this workgroup's piece of it, is finished ----
        int elane = lane;
        asm volatile("" : "+v"(elane));   // opaque: the addresses below are formed here, not kept across the loop
        if (seg_kb == 0 && kb == p.nk) {
            // (a short segment: the norms may still be on their way)
            if (seg_steps <= NS + 4) wait_global_loads_le<0>();
            f32x4 nrm[C::EB];
            const f32x4 *nb = reinterpret_cast<const f32x4 *>(smem + NORMS + (par * 8 + w) * 256);
#pragma unroll
            for (int i = 0; i < C::EB; ++i) nrm[i] = nb[i * 4 + (elane >> 4)];
            emit_tile<C>(acc, nrm, p, mt, nt, we, wq, elane);
            since = p.projection ? NS : 1;   // (a projection's stores are not counted)
        } else {
            // slot 0: the piece that does not hold the tile's first k-step, slot 1: the one that does
            f32x4 *dst = reinterpret_cast<f32x4 *>(p.partial) +
                         ((size_t)blockIdx.x * 2 + (seg_kb == 0 ? 1 : 0)) * (size_t)(C::BM * kTileN / 4) + elane;
#pragma unroll
            for (int i = 0; i < C::EB; ++i)
#pragma unroll
                for (int j = 0; j < C::QB; ++j) dst[((w * C::EB + i) * C::QB + j) * 64] = acc[i][j];
            since = NS;   // (ordinary stores, straight from the matrix results: the waits take none of them for granted)
        }
        clear();
        seg_steps = 0;
        seg_kb = 0;
        kb = 0;
        par ^= 1;
        if (++nt == p.n_tiles) {
            nt = 0;
            ++mt;
        }
    }
    wait_global_loads_le<0>();   // the refills past the end land before the workgroup gives its LDS back
}

// The tiles cut by the ends of ranges: add up the pieces, then emit.  Block (x, w): wave part w of tile x (BY_TILE), or of the
// tile whose first k-step, but not its last, lies in range x, where there are fewer ranges than tiles.  (By range, tiles of
// 2^m k-steps begin in ranges that are all on one XCD: 64 queries, 4,000 x 8,192: 48 us of a look-up of 90, which takes 50 by
// tile; 128 inputs 8,192 -> 1,024 38 -> 20.)  Its four waves take a quarter of the pieces each, in the
// order of the ranges, and the first adds the quarters up in order (one wave reading the 128 pieces of a
// 32,768-value projection one after the other took 70 us).
template <class C, bool BY_TILE>
__global__ __launch_bounds__(256) void stream_fixup_kernel(StreamArgs p)
{
    __shared__ f32x4 part[3][C::EB * C::QB][64];
    const int nq = p.count ? *p.count : p.b;
    const int live_mt = (nq + C::BM - 1) / C::BM;
    const int64_t total = (int64_t)live_mt * p.n_tiles * p.nk;
    const int range = BY_TILE ? (int)((int64_t)blockIdx.x * p.nk / p.len) : (int)blockIdx.x;
    const int64_t g0 = (int64_t)range * p.len;
    if ((BY_TILE ? (int64_t)blockIdx.x * p.nk : g0) >= total) return;
    const int64_t g1 = g0 + p.len < total ? g0 + p.len : total;
    const int64_t tile = BY_TILE ? (int64_t)blockIdx.x : (g1 - 1) / p.nk;
    const int64_t t0 = tile * p.nk, t1 = t0 + p.nk;
    // uniform: the tile lies in the range, or (by range) the range's last tile starts earlier
    if (BY_TILE ? g1 >= t1 : g1 == t1 || t0 < g0) return;
    const int w = blockIdx.y, lane = threadIdx.x & 63;
    const int v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int we = w % C::WE, wq = w / C::WE;
    const int pieces = (int)((t1 - 1) / p.len) - range + 1;
    f32x4 acc[C::EB][C::QB];
#pragma unroll
    for (int i = 0; i < C::EB; ++i)
#pragma unroll
        for (int j = 0; j < C::QB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const size_t piece = (size_t)(C::BM * kTileN / 4);
    const f32x4 *src = reinterpret_cast<const f32x4 *>(p.partial) + (size_t)w * C::EB * C::QB * 64 + lane;
#pragma unroll 2
    for (int n = pieces * v / 4; n < pieces * (v + 1) / 4; ++n) {
        // the first piece is its range's slot 1, the others are slot 0 of theirs
        const f32x4 *s0 = src + ((size_t)(range + n) * 2 + (n == 0 ? 1 : 0)) * piece;
#pragma unroll
        for (int i = 0; i < C::EB; ++i)
#pragma unroll
            for (int j = 0; j < C::QB; ++j) {
                const f32x4 x = s0[(i * C::QB + j) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += x[e];
            }
    }
    if (v > 0) {
#pragma unroll
        for (int i = 0; i < C::EB; ++i)
#pragma unroll
            for (int j = 0; j < C::QB; ++j) part[v - 1][i * C::QB + j][lane] = acc[i][j];
    }
    __syncthreads();
    if (v > 0) return;
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int i = 0; i < C::EB; ++i)
#pragma unroll
            for (int j = 0; j < C::QB; ++j) {
                const f32x4 x = part[u][i * C::QB + j][lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] += x[e];
            }
    const int mt = (int)(tile / p.n_tiles), nt = (int)(tile % p.n_tiles);
    f32x4 nrm[C::EB];
#pragma unroll
    for (int i = 0; i < C::EB; ++i)
        nrm[i] = *reinterpret_cast<const f32x4 *>(p.norm + (size_t)nt * kTileN + we * C::EB * 16 + i * 16 + (lane >> 4) * 4);
    emit_tile<C>(acc, nrm, p, mt, nt, we, wq, lane);
}

template <class C>
hipError_t launch_cfg(const DistPlan &pl, const DistArgs &a, hipStream_t s)
{
    StreamArgs k{};
    k.q_bf = a.q_bf;
    k.c_bf = a.c_bf;
    k.norm = a.norm;
    k.keys = a.keys;
    k.bmin = a.bmin;
    k.partial = a.partial;
    k.count = a.count;
    k.b = a.b;
    k.n_tiles = pl.n_tiles;
    k.nk = a.d_pad / kKB;
    k.len = pl.st_len;
    k.n_pad = (int64_t)pl.n_tiles * kTileN;
    k.once = pl.m_tiles == 1 && !a.projection;   // (weights are small and stay in the caches)
    k.projection = a.projection ? 1 : 0;
    k.relu = a.relu ? 1 : 0;
    k.n = a.n;
    k.ld = a.projection ? a.ld : k.n_pad;
    hipLaunchKernelGGL((dist_stream_kernel<C>), dim3((unsigned)pl.st_wgs), dim3(512), 0, s, k);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !pl.st_cut) return e;
    const int64_t tiles = (int64_t)pl.m_tiles * pl.n_tiles;
    if (tiles <= pl.st_wgs) hipLaunchKernelGGL((stream_fixup_kernel<C, true>), dim3((unsigned)tiles, 8), dim3(256), 0, s, k);
    else hipLaunchKernelGGL((stream_fixup_kernel<C, false>), dim3((unsigned)pl.st_wgs, 8), dim3(256), 0, s, k);
    return hipGetLastError();
}

}  // namespace

// Query tile and ranges of the streaming kernel.
DistPlan plan_stream(int64_t b, int64_t n, int r, int num_cus, int64_t d_pad, StreamCut cut)
{
    DistPlan pl{};
    pl.variant = 4;
    pl.r = r;
    pl.n_tiles = (int)((n + kTileN - 1) / kTileN);
    pl.num_cus = num_cus;
    pl.n_splits = pl.alloc_splits = 1;
    pl.max_splits = pl.n_tiles;
    const int nk = (int)(d_pad / kKB);
    const int wgs = 2 * num_cus;
    int bm = b <= 16 ? 16 : (b <= 32 ? 32 : (b <= 64 ? 64 : 128));
    auto total = [&](int m) { return ((b + m - 1) / m) * (int64_t)pl.n_tiles * nk; };
    // a small cache: smaller query tiles give more workgroups something to do (the cache, re-read per
    // query tile, sits in L2): 256 queries x 2,000 x 512, 52 us with one 256-row tile per cache tile (8
    // workgroups), 36 us with 16 x 8 tiles
    while (bm > 16 && total(bm) < 8 * (int64_t)wgs) bm >>= 1;
    pl.bm = bm;
    pl.m_tiles = (int)((b + bm - 1) / bm);
    if (pl.m_tiles < 1) pl.m_tiles = 1;
    pl.b_pad = (int64_t)pl.m_tiles * bm;
    const int64_t all = (int64_t)pl.m_tiles * pl.n_tiles * nk;
    int64_t len = (all + wgs - 1) / wgs;
    // at least 8 k-steps a workgroup, 16 where a cut tile's slot is 128 KiB
    const int64_t least = bm == 128 ? 16 : 8;
    if (len < least) len = least;
    // whole tiles where a tile is short (a second launch costs more than the idle workgroups) or where a
    // range holds so many that cutting one gains little
    bool whole = cut == StreamCut::none || nk <= 32 || len >= 16 * (int64_t)nk;
    if (cut == StreamCut::where_faster && !whole) {
        // Whole tiles go in rounds of wgs tiles, nk k-steps each, of which the last may leave most of the chip idle; a
        // cut evens the ranges out and costs the slots and stream_fixup_kernel. A round's k-step takes 0.45 us by its
        // latency for each workgroup of the fullest CU, or 2.6 ns for each tile (16 KiB at 6.3 TB/s) where
        // memory is what bounds it; the fix-up 6 us and 0.1 us for each 128-query tile among the first wgs. Fitted to
        // the times of both at 260 random shapes (257 .. 374,631 rows, 1,025 .. 65,536 columns, up to 200 queries):
        // always cut 39.6 ms in sum, by this line 38.04, the faster of the two at each shape 38.00.
        //   99,862 x 1,585, 74 queries: cut 183 us, whole 103. 374,631 x 3,582, 92 queries: 717, 577.
        //   78,855 x 16,887, 15 queries: cut 460 us, whole 517. 9,050 x 33,202, 12 queries: 166, 395.
        const double tiles = (double)pl.m_tiles * pl.n_tiles, rounds = std::ceil(tiles / wgs);
        const double last = tiles - (rounds - 1) * wgs;
        auto round_us = [&](double t) { return nk * std::max(std::ceil(t / num_cus) * 0.45, t * 0.0026); };
        const double t_whole = (rounds - 1) * round_us(wgs) + round_us(last);
        const double t_cut = std::max(tiles * nk * 0.0026, (double)len * 0.45) + 6.0 + 0.1 * std::min(tiles, (double)wgs) * bm / 128;
        whole = t_whole <= t_cut;
    }
    if (whole) len = (len + nk - 1) / nk * nk;
    pl.st_len = len;
    pl.st_wgs = (int)((all + len - 1) / len);
    pl.st_cut = len % nk != 0;
    return pl;
}

hipError_t launch_dist_stream(const DistPlan &pl, const DistArgs &a, hipStream_t s)
{
    if (pl.variant != 4 || pl.st_wgs < 1 || pl.st_len < 1 || a.d_pad < 64 || a.d_pad % kPadD != 0 || !a.keys || (!a.bmin && !a.projection) || (a.projection && a.ld < a.n) || a.b < 1 ||
        a.b > pl.b_pad || (pl.st_cut && !a.partial))
        return hipErrorInvalidValue;
    switch (pl.bm) {
    case 16: return launch_cfg<StreamCfg<16, 1, 4>>(pl, a, s);
    case 32: return launch_cfg<StreamCfg<32, 1, 4>>(pl, a, s);
    case 64: return launch_cfg<StreamCfg<64, 1, 3>>(pl, a, s);
    case 128: return launch_cfg<StreamCfg<128, 2, 3>>(pl, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace fz
