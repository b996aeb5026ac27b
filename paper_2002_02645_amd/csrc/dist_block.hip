// Distance pass for batches: block minima instead of candidate lists.
//
// The fused kernel folds every 256 x 256 tile of keys into per-query lists in LDS.  That takes 12 us a
// tile once the lists have settled and 60 us for a workgroup's first one, whatever the activation's
// length; a tile's matrix work takes 11 us at 512 values (4,096 queries x 50,000 x 512: 399 us for 140 us
// of matrix work).  Here a tile leaves one number per query and block of eight entries, the smallest key
// of the block (4 bytes per 8 entries and query), and nothing in the kernel depends on the data: four
// max3 per block in registers, one 8-byte store per two blocks, no LDS, no barrier.  block_finish_kernel
// then finds the R blocks with the smallest minima, which hold the R best entries by the coarse key
// and more, and re-scores their 8 R entries exactly.  That is cheap for short rows and few queries.  Elsewhere
// (block_next_pays in the API file) a block leaves 16 bits more: which entry has the smallest key, and by how
// much it leads (block_next), and one row per block is re-scored.  That takes some 25 instructions per block in place of
// five, 2.4 us a tile (4,096 x 50,000 x 512: 189 -> 209 - 220 us here, 141 -> 73 in the finishing kernel).
//
//   - The accumulators start at -|c|^2 / 2 (the first matrix instruction of a tile takes the norms as its
//     third operand), so a finished accumulator is q.c - |c|^2 / 2 = -key / 2: no arithmetic on the way out
//     but the maximum and an exact scaling by -2.
//   - The matrix instruction takes entries as its rows and queries as its columns: a lane holds four
//     consecutive entries of one query per instruction, and a block is the lane's eight entries of two
//     instructions 16 entries apart, so that its maximum needs no other lane.
//   - 8 waves (2 x 4), each 128 queries x 64 entries, the k-step in two halves as in the batched kernel's
//     8-wave loop; the ring of four stages runs on from one tile to the next (a tile has as few as two
//     k-steps), so a tile costs no prologue and no drain.  Loads and stores are counted by the kernel.
//   - Work: whole tiles, dealt evenly and contiguously to one workgroup per CU in the order (group of
//     query tiles, cache tile, query tile of the group): a workgroup uses a cache tile for all query tiles
//     of a group in a row, and a group's queries (1 or 2 MB) stay in the XCD's L2.
//
// 4,096 x 50,000 x 512, k = 10: whole look-ups 503 us with lists, 327 with minima alone, 286 with the further bits (where the
// first blocks confirm more of the queries 493, 292, 280); 300 queries 172, 62, 62 us; 20,011 x 517 fp32, 1,537 queries, k = 20
// 320, 189, 102.
//
// Paper: Sec. 3 (k nearest neighbours), Sec. 4 "Computational Complexity".
#include "freeze_internal.h"
#include "select_common.h"

#include <type_traits>

namespace fz {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

namespace {

constexpr int kStageHalf = kTileN * kKB * 2;    // 16 KiB: one k-block of 256 rows
constexpr int kStageBytes = 2 * kStageHalf;     // queries, then entries
constexpr int NS = 4;                           // stages
constexpr int LPS = 4, LB = 2;                  // loads per wave and stage; issued in the half-step that frees the stage
constexpr int AM = 8, AH = 4, BNB = 4;          // 16-query blocks per wave (and half), 16-entry blocks per wave
constexpr int kNorms = NS * kStageBytes;        // byte offset of the norm buffers: per tile parity and wave, 64 floats
constexpr int kLds = kNorms + 2 * 8 * 256;
static_assert(kLds <= 163840, "LDS budget");

struct BlockArgs {
    const uint16_t *q_bf;   // tiled, tiles of 256 rows
    const uint16_t *c_bf;
    const float *norm;
    float *bkey;            // [b_pad, n_pad / 8] smallest key of every block
    uint32_t *bnext;        // [b_pad, n_pad / 16] of every block: where it lies, and a bound of the others (block_next in select_common.h)
    const int32_t *count;   // device: live queries, or null (= b)
    int b, n_tiles, nk, group;   // nk k-steps per tile (even); group: query tiles that share a cache tile in a row
};

// (one instruction each, without the compiler's quieting of signalling NaNs, which no arithmetic leaves)
#define FZ_OP3(name, op)                                                             \
    __device__ __forceinline__ float name(float a, float b, float c)                 \
    {                                                                                \
        float r;                                                                     \
        asm(op " %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));                \
        return r;                                                                    \
    }
FZ_OP3(max3, "v_max3_f32")
FZ_OP3(med3, "v_med3_f32")
#undef FZ_OP3
#define FZ_OP2(name, op)                                                             \
    __device__ __forceinline__ float name(float a, float b)                          \
    {                                                                                \
        float r;                                                                     \
        asm(op " %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));                            \
        return r;                                                                    \
    }
FZ_OP2(max2, "v_max_f32")
FZ_OP2(min2, "v_min_f32")
#undef FZ_OP2

// The largest of the eight values of a block and, in 16 bits, its place and its lead over the second largest.
template <bool NEXT>
__device__ __forceinline__ float block_top(const f32x4 &a, const f32x4 &b, uint32_t &next)
{
    const float m0 = max3(a[0], a[1], a[2]), m1 = max3(a[3], b[0], b[1]), m2 = max2(b[2], b[3]);
    if constexpr (!NEXT) return max3(m0, m1, m2);
    const float s0 = med3(a[0], a[1], a[2]), s1 = med3(a[3], b[0], b[1]), s2 = min2(b[2], b[3]);
    const float top = max3(m0, m1, m2);
    const float second = max2(med3(m0, m1, m2), max3(s0, s1, s2));
    uint32_t at = 0;
#pragma unroll
    for (int e = 1; e < 8; ++e) at = (e < 4 ? a[e & 3] : b[e & 3]) == top ? e : at;
    next = block_next(top - second, at);
    return top;
}

// NEXT: 16 more bits per block (block_next)
template <bool NEXT>
__global__ __launch_bounds__(512) void dist_block_kernel(BlockArgs p)
{
    constexpr int STORES = NEXT ? 2 * AM : AM;      // per wave and tile
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLds];
    const bf16x8 *smem16 = reinterpret_cast<const bf16x8 *>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 2, wn = w & 3;
    const int nq = p.count ? *p.count : p.b;
    const int live_mt = (nq + 255) / 256;
    const int64_t tiles = (int64_t)live_mt * p.n_tiles;
    // contiguous shares, neighbouring shares on one XCD (block id modulo 8)
    const int W = (int)gridDim.x, x8 = blockIdx.x & 7, a8 = W >> 3, rem8 = W & 7;
    const int xid = x8 * a8 + (x8 < rem8 ? x8 : rem8) + ((int)blockIdx.x >> 3);
    const int64_t t0 = tiles * xid / W, t1 = tiles * (xid + 1) / W;
    if (t0 >= t1) return;   // uniform
    const int steps = (int)(t1 - t0) * p.nk;

    // cursor over (tile, k-step): tile t = ((query tile group, cache tile), query tile of the group)
    struct Cursor {
        int g0, gn, mt, nt, kb;   // first query tile and size of the group, query tile, cache tile, k-step
    };
    auto cursor_at = [&](int64_t t) {
        Cursor c;
        const int64_t per_group = (int64_t)p.group * p.n_tiles;
        const int g = (int)(t / per_group);
        const int64_t r = t - g * per_group;
        c.g0 = g * p.group;
        c.gn = live_mt - c.g0 < p.group ? live_mt - c.g0 : p.group;
        c.nt = (int)(r / c.gn);
        c.mt = c.g0 + (int)(r - (int64_t)c.nt * c.gn);
        c.kb = 0;
        return c;
    };
    auto next_tile = [&](Cursor &c) {
        c.kb = 0;
        if (++c.mt == c.g0 + c.gn) {
            c.mt = c.g0;
            if (++c.nt == p.n_tiles) {
                c.nt = 0;
                c.g0 += c.gn;
                c.gn = live_mt - c.g0 < p.group ? live_mt - c.g0 : p.group;
                c.mt = c.g0;
            }
        }
    };
    Cursor cur = cursor_at(t0), ld = cur;
    int ld_left = steps;    // the loads' cursor stops at the last k-step, which the refills past the end repeat
    auto advance = [&]() {
        if (ld_left > 1) {
            --ld_left;
            if (++ld.kb == p.nk) next_tile(ld);
        }
    };
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
    const uint32_t lane_off = w * 1024 + lane * 16;
    const uint64_t qbase = (uint64_t)(uintptr_t)p.q_bf, cbase = (uint64_t)(uintptr_t)p.c_bf;
    // load l of the stage at the loads' cursor: two of queries, two of entries, 8 KiB of the workgroup each
    auto issue_one = [&](int stage, int l) {
        const uint64_t src = l < 2 ? uniform_u64(qbase + ((uint64_t)ld.mt * p.nk + ld.kb) * kStageHalf)
                                   : uniform_u64(cbase + ((uint64_t)ld.nt * p.nk + ld.kb) * kStageHalf);
        load16_global_to_lds(src + (l & 1) * 8192, lane_off, smem_base + stage * kStageBytes + w * 1024 + l * 8192);
    };
    auto issue_norms = [&](int nt, int par) {
        const uint64_t src = uniform_u64((uint64_t)(uintptr_t)(p.norm + (size_t)nt * kTileN + wn * 64));
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(smem_base + kNorms + (par * 8 + w) * 256), "v"(lane * 4), "s"(src)
                     : "memory", "m0");
    };

    const int rowA = wm * 128 + (lane & 15), rowB = wn * 64 + (lane & 15);
    const int rdA = rowA * 4 + ((lane >> 4) ^ tiled_chunk_swizzle(rowA));
    const int rdB = kStageHalf / 16 + rowB * 4 + ((lane >> 4) ^ tiled_chunk_swizzle(rowB));
    bf16x8 af[2][AH], bfr[2][BNB];
    auto read_a = [&](int h, int stage, int i) { af[h][i] = smem16[stage * (kStageBytes / 16) + rdA + (h * AH + i) * 64]; };
    auto read_b = [&](int set, int stage, int j) { bfr[set][j] = smem16[stage * (kStageBytes / 16) + rdB + j * 64]; };
    f32x4 acc[AM][BNB], nrm[BNB];
    // accumulator starts of the tile whose norms lie in buffer `par`: -|c|^2 / 2 (padding entries: -inf)
    auto read_norms = [&](int par) {
        const f32x4 *src = reinterpret_cast<const f32x4 *>(smem + kNorms + (par * 8 + w) * 256);
#pragma unroll
        for (int j = 0; j < BNB; ++j) {
            const f32x4 v = src[j * 4 + (lane >> 4)];
#pragma unroll
            for (int e = 0; e < 4; ++e) nrm[j][e] = -0.5f * v[e];
        }
    };

    int par = 0, stores_at = NS;   // stores_at: k-steps since the last tile's stores
    issue_norms(cur.nt, 0);
#pragma unroll
    for (int ps = 0; ps < NS; ++ps) {
#pragma unroll
        for (int l = 0; l < (ps == NS - 1 ? LB : LPS); ++l) issue_one(ps, l);
        if (ps < NS - 1) advance();
    }
    wait_global_loads_le<(NS - 2) * LPS + LB>();
    __syncthreads();
    read_norms(0);
#pragma unroll
    for (int i = 0; i < AH; ++i) read_a(0, 0, i);
#pragma unroll
    for (int j = 0; j < BNB; ++j) read_b(0, 0, j);

    int st = 0;
    // The k-step of the batched kernel's 8-wave loop: half the wave's query blocks against all its entry
    // blocks, then, past the step's only barrier, the other half.  The second half's A fragments are read
    // during the first half; the next stage's first fragments and the refill of the stage just freed leave
    // between the second half's matrix instructions, the rest of the refill between the next step's first ones.  Matrix
    // instructions in a row share their first operand: a register-only loop of 4 x 8 blocks sustains 2,140 TFLOP/s so and 2,020
    // where they share the second (one wave per SIMD, power limit).
    auto k_step = [&](auto set_tag, auto first_tag) {
        constexpr int set = decltype(set_tag)::value;
        constexpr bool first = decltype(first_tag)::value;   // the tile's first k-step: the accumulators start at the norms
        const int nst = (st + 1 == NS) ? 0 : st + 1;
        const int pst = (st == 0) ? NS - 1 : st - 1;
#pragma unroll
        for (int i = 0; i < AH; ++i) read_a(1, st, i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < BNB; ++j) {
#pragma unroll
            for (int t = 0; t < AH; ++t) {
                const int i = j & 1 ? AH - 1 - t : t;
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[set][j], af[0][i], first ? nrm[j] : acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int l = LB + j * (LPS - LB) / BNB; l < LB + (j + 1) * (LPS - LB) / BNB; ++l) issue_one(pst, l);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance();
        // own part of the next k-block has landed; younger than it are NS - 2 stages and, for NS - 2 steps
        // after a tile's end, that tile's stores
        if (stores_at <= NS - 2) wait_global_loads_le<(NS - 2) * LPS + STORES>();
        else wait_global_loads_le<(NS - 2) * LPS>();
        ++stores_at;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();                                // ... everyone's; and stage st is free
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < BNB; ++j) {
#pragma unroll
            for (int t = 0; t < AH; ++t) {
                const int i = j & 1 ? AH - 1 - t : t;
                acc[AH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[set][j], af[1][i], first ? nrm[j] : acc[AH + i][j], 0, 0, 0);
            }
#pragma unroll
            for (int rr = j * 8 / 3; rr < (j + 1) * 8 / 3 && rr < AH + BNB && j < 3; ++rr) {
                if (rr < AH)
                    read_a(0, nst, rr);
                else
                    read_b(set ^ 1, nst, rr - AH);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int l = j * LB / BNB; l < (j + 1) * LB / BNB; ++l) issue_one(st, l);
            __builtin_amdgcn_sched_barrier(0);
        }
        st = nst;
    };
    using S0 = std::integral_constant<int, 0>;
    using S1 = std::integral_constant<int, 1>;

    for (int64_t t = t0; t < t1; ++t) {
        // the next tile's norms, older than every stage in flight when they are read
        Cursor nxt = cur;
        next_tile(nxt);
        if (t + 1 < t1) issue_norms(nxt.nt, par ^ 1);
        k_step(S0{}, std::true_type{});
        k_step(S1{}, std::false_type{});
        for (int kb = 2; kb < p.nk; kb += 2) {
            k_step(S0{}, std::false_type{});
            k_step(S1{}, std::false_type{});
        }
        // ---- the tile is finished: the block minima ----
        if (p.nk <= 6) wait_global_loads_le<0>();   // a short tile: the next one's norms may still be on their way
        int elane = lane;
        asm volatile("" : "+v"(elane));   // opaque: the addresses are formed here, not kept across the loop
        // (the compiler does not see that max3 reads matrix results: the no-ops are the distance the hardware
        // wants.  They take the first half of the accumulators through their operands and lie between two
        // statements that take the second half: every matrix instruction of the tile comes before them and every
        // maximum after, by the values alone, wherever the compiler moves either.)
        auto second_half = [&]() {
            asm volatile(""
                         : "+v"(acc[4][0]), "+v"(acc[4][1]), "+v"(acc[4][2]), "+v"(acc[4][3]),
                           "+v"(acc[5][0]), "+v"(acc[5][1]), "+v"(acc[5][2]), "+v"(acc[5][3]),
                           "+v"(acc[6][0]), "+v"(acc[6][1]), "+v"(acc[6][2]), "+v"(acc[6][3]),
                           "+v"(acc[7][0]), "+v"(acc[7][1]), "+v"(acc[7][2]), "+v"(acc[7][3]));
        };
        second_half();
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7"
                     : "+v"(acc[0][0]), "+v"(acc[0][1]), "+v"(acc[0][2]), "+v"(acc[0][3]),
                       "+v"(acc[1][0]), "+v"(acc[1][1]), "+v"(acc[1][2]), "+v"(acc[1][3]),
                       "+v"(acc[2][0]), "+v"(acc[2][1]), "+v"(acc[2][2]), "+v"(acc[2][3]),
                       "+v"(acc[3][0]), "+v"(acc[3][1]), "+v"(acc[3][2]), "+v"(acc[3][3]));
        second_half();
        const int64_t nb = (int64_t)p.n_tiles * (kTileN / 8);
        const int64_t at = ((int64_t)cur.mt * 256 + wm * 128 + (elane & 15)) * nb + cur.nt * (kTileN / 8) + wn * 8 + (elane >> 4) * 2;
        float *dst = p.bkey + at;
        uint32_t *dst_next = p.bnext + (at >> 1);
#pragma unroll
        for (int i = 0; i < AM; ++i) {
            f32x2 v;
            uint32_t nx[2];
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) v[j2] = -2.f * block_top<NEXT>(acc[i][2 * j2], acc[i][2 * j2 + 1], nx[j2]);
            // (rows past the batch are written too: the buffer has whole tiles of rows)
            asm volatile("global_store_dwordx2 %0, %1, off" ::"v"(dst + i * 16 * nb), "v"(v) : "memory");
            if constexpr (NEXT) asm volatile("global_store_dword %0, %1, off" ::"v"(dst_next + i * 8 * nb), "v"(nx[0] | nx[1] << 16) : "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
        if (t + 1 < t1) read_norms(par ^ 1);
        stores_at = 1;
        cur = nxt;
        par ^= 1;
    }
    wait_global_loads_le<0>();   // the refills past the end land before the workgroup gives its LDS back
}

}  // namespace

DistPlan plan_block(int64_t b, int64_t n, int r, int num_cus, int64_t d_pad, bool next)
{
    DistPlan pl{};
    pl.variant = 5;
    pl.next = next;
    pl.bm = 256;
    pl.r = r;
    pl.m_tiles = (int)((b + 255) / 256);
    if (pl.m_tiles < 1) pl.m_tiles = 1;
    pl.n_tiles = (int)((n + kTileN - 1) / kTileN);
    pl.n_splits = pl.alloc_splits = 1;
    pl.max_splits = pl.n_tiles;
    pl.num_cus = num_cus;
    pl.b_pad = (int64_t)pl.m_tiles * 256;
    const int64_t tiles = (int64_t)pl.m_tiles * pl.n_tiles;
    pl.grid_units = (int)(tiles < num_cus ? tiles : num_cus);
    // query tiles of a group: their bf16 rows take at most a quarter of an XCD's 4 MB of L2 (10,000 x 50,000 x
    // 512: 676 us at 1 MB, 701 at 2, 728 at 4)
    const int64_t tile_bytes = 256 * d_pad * 2;
    // ... at 2 MB where the cache exceeds the memory-side cache (256 MB) and every group reads it from HBM again (640 x
    // 520,980 x 1,100: 988 us at 1 MB, 832 at 2)
    const int64_t cache_bytes = (int64_t)pl.n_tiles * kTileN * d_pad * 2;
    int64_t g = (cache_bytes > ((int64_t)256 << 20) ? 2 << 20 : 1 << 20) / tile_bytes;
    g = g < 1 ? 1 : g;
    pl.group = (int)(g < pl.m_tiles ? g : pl.m_tiles);
    return pl;
}

hipError_t launch_dist_block(const DistPlan &pl, const DistArgs &a, hipStream_t s)
{
    if (pl.variant != 5 || !a.keys || (pl.next && !a.bnext) || a.d_pad < 64 || a.d_pad % kPadD != 0 || a.b < 1 || a.b > pl.b_pad || pl.group < 1 || pl.grid_units < 1)
        return hipErrorInvalidValue;
    BlockArgs k{a.q_bf, a.c_bf, a.norm, a.keys, a.bnext, a.count, a.b, pl.n_tiles, a.d_pad / kKB, pl.group};
    if (pl.next) hipLaunchKernelGGL(dist_block_kernel<true>, dim3((unsigned)pl.grid_units), dim3(512), 0, s, k);
    else hipLaunchKernelGGL(dist_block_kernel<false>, dim3((unsigned)pl.grid_units), dim3(512), 0, s, k);
    return hipGetLastError();
}

}  // namespace fz
