// Matrix product of many fp32 rows with a few hundred prepared ones, the fp32 rows converted on their way into the
// matrix cores (gfx950 / CDNA4).  It serves the assignment step of the k-means build and the projection.
//
// k-means.
// The assignment needs, for every point, the nearest of a few hundred centres.  Through the look-up that was a bf16
// copy of the points (read and written once per build), a bf16 pass with candidate lists and eight exactly re-scored
// fp32 centres per point: 50,000 x 8,192, 200 centres 250 + 820 us a round, the latter for 13 GB of centre rows
// out of the L2s, and 430 us for the copy.  Here a value x is taken as hi + lo, two bf16 values, and
//     q.c = hi.hi + hi.lo + lo.hi   (lo.lo, at most 2^-16 of the product, is left out)
// so that the keys are good to 2^-12 of |q||c|, mostly far better, instead of 2^-7 and most points' nearest
// centre is known from them alone (kmeans_pick_kernel, which re-scores what the bound of key_error leaves open).
// Three matrix instructions per block instead of one: 0.51 TFLOP in that case, 400 to 470 us (1.1 to 1.25 PFLOP/s; the matrix
// pipes are busy 60 % of the time at 2.0 GHz, and it is the power limit that sets the clock), and 90 to 115 us for the choice, which
// re-scores a tenth of the points.  The whole build, two rounds, 4,710 -> 2,240 us; 50,000 x 512 1,590 -> 437, 50,000 x 8,191
// 6,810 -> 2,640, 50,000 x 8,192 with 400 centres 5,680 -> 3,600, 3,000 x 300 with 20 centres 232 -> 152.
// (Sums cut at half the length, with half the error: 70 us for the choice, 25 more for the product, 2,195.)
//
//   - 512 threads, 4 x 2 waves, a wave 64 rows x half the columns; a k-step is 32 elements.  The fp32 rows are copied
//     as they are (LDS-direct loads, ring of three stages: the stage after the next is on its way for one and a
//     half k-steps before it is needed), and a wave converts its 64 rows' fragments of the next k-step between the matrix
//     instructions of this one.  Converting before the LDS would need the loads in registers; a prepared copy
//     would need the memory traffic this kernel is there to save.
//   - The prepared rows (hi and lo, tiled like a cache) come out of L2 one k-step ahead, two stages.
//   - LDS: 3 x 32 KiB + 2 x 2 KiB per 16 columns, one workgroup per CU.  A k-step of 13 column blocks reads 164 KiB of
//     fragments (about half the time of its matrix instructions) and writes 58.
//   - Work: the flattened (row tile, column tile, k-step) space in even ranges, one per CU (196 row tiles would leave
//     60 CUs idle); a range leaves the sums of each tile it touches in a slot, and the reader of the sums adds the
//     slots of a tile in order.  Many tiles per CU: whole tiles, one slot.
//
// Projection: one bf16 value per element on both sides, as the layer is defined.  A bf16 copy of the inputs first cost 82 us
// at 10,000 x 8,192 -> 1,024 (and the product 148, the sums of cut tiles 36).
//   - Ranges of the (row tile, k-step) space, each for a group of workgroups of one XCD, one per column tile: they take the
//     same fp32 rows at about the same time, out of HBM once and out of the XCD's L2 for the others.  (What is left of the XCDs'
//     workgroups forms groups across them: 5 of 85 with three column tiles.)
//   - Bound by what reaches the CUs out of L2, 48 KiB per k-step and workgroup, at 10 TB/s: 195 us there for 168 GFLOP (0.86
//     PFLOP/s).  Whole calls 265 -> 209 us; 10,000 x 32,768 -> 256 604 -> 319; 10,000 x 1,000 -> 1,500 75 -> 41; 300 x 30,000 ->
//     300 176 -> 35; 1,500 x 8,192 -> 1,024 87 -> 59 (47 with the longer sums that plan_projection no longer takes).
//
// Paper: Sec. 4 "k-means"; Sec. 3 (one-layer dimensionality reduction).
#include "freeze_internal.h"
#include "select_common.h"

#include <algorithm>
#include <type_traits>

namespace fz {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

namespace {


// LDS-direct 4-byte load: as load16_global_to_lds, 4 bytes per lane
__device__ __forceinline__ void load4_global_to_lds(uint64_t sbase, uint32_t voff, uint32_t lds_byte_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_byte_addr), "v"(voff), "s"(sbase)
                 : "memory", "m0");
}

struct RowsGemmArgs {
    const float *x;               // [n, d]
    const uint16_t *hi, *lo;      // prepared rows, tiled (tiles of kTileN rows, d_pad elements); lo: split ones only
    float *part;                  // [tile][slot][kRowsTile][16 NCB]
    float *sq;                    // [row tile][slot][kRowsTile] sums of squares of the fp32 rows (split ones)
    int64_t n, d, d_pad;
    int64_t len;                  // k-steps of a range
    int nk, n_tiles, m_tiles, slots;
    // projection
    int rows;                     // per tile
    int groups;                   // per XCD: n_tiles workgroups of one XCD share the fp32 rows of a range
    const float *bias;            // [n_tiles 16 NCB at least]
    float *out;                   // [n, m]
    int64_t m;
    int relu;
};

// four consecutive columns of one output row of the projection
__device__ __forceinline__ void store_projected(const RowsGemmArgs &p, int64_t row, int64_t col, f32x4 v)
{
    const f32x4 b = *reinterpret_cast<const f32x4 *>(p.bias + col);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] += b[e];
        if (p.relu) v[e] = __builtin_fmaxf(v[e], 0.f);
    }
    float *dst = p.out + row * p.m + col;
    if (p.m % 4 == 0) {   // uniform; col is a multiple of 4, so no group of four crosses the end
        if (col < p.m) *reinterpret_cast<f32x4 *>(dst) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (col + e < p.m) dst[e] = v[e];
    }
}

__device__ __forceinline__ int a_swizzle(int row)
{
    const int u = (row >> 1) & 7;
    return u ^ (((u + 2) & 4) >> 1);
}

// VEC: rows start on 16-byte boundaries (d a multiple of 4)
// NCB: blocks of 16 columns of a tile; the second wave of a row of waves has one less where the number is odd
// SPLIT: hi + lo on both sides (k-means); else one bf16 value on both sides, and the sums of a tile that no range's end
// cuts go straight to the output (projection)
// RB: blocks of 16 rows of a wave (SPLIT: 4)
template <int NCB, bool VEC, bool SPLIT, int RB>
__global__ __launch_bounds__(512) void rows_gemm_kernel(RowsGemmArgs p)
{
    constexpr int TNB = (NCB + 1) / 2;                  // column blocks of a wave
    constexpr int NC = 16 * NCB;                        // columns of a tile
    constexpr int B_IMG = NC * 64;                      // one k-step of hi (or lo)
    constexpr int B_STAGE = SPLIT ? 2 * B_IMG : B_IMG;
    // groups of matrix instructions that the prepared rows' fragments are read ahead: a group is 12 or 4 of them
    constexpr int PD = SPLIT ? 1 : 2, RING = SPLIT ? 2 : 4;
    static_assert((2 * TNB) % RING == 0 && TNB > PD, "fragments' register sets");
    // A k-step of the projection has a third of the matrix work, and its prepared rows come from beyond L2 (the groups of an
    // XCD are at different depths).  As many stages of both as fit, so that loads leave one k-step ahead with tiles of 256 rows,
    // two with 192; plan_projection chooses.
    constexpr int ROWS = 64 * RB;                       // rows of a tile
    static_assert(!SPLIT || ROWS == kRowsTile, "");
    constexpr int kAStages = RB == 4 ? 3 : 4, kAStage = ROWS * kKB * 4;   // one k-step of the fp32 rows
    constexpr int NSB = SPLIT ? 2 : kAStages;
    constexpr int NBI = B_STAGE / 1024;                 // load instructions of a stage
    constexpr int NI_B = (NBI + 7) / 8;                 // per wave (the last wave's surplus repeats a load)
    constexpr int NI_A = VEC ? RB : 4 * RB;
    constexpr int WR = ROWS / 8;                        // rows a wave loads
    // loads younger than those a step waits for
    constexpr int AHEAD = SPLIT ? NI_A : (NSB - 2) * (NI_A + NI_B);
    constexpr int NL = NI_B + NI_A;
    constexpr int kB = kAStages * kAStage;              // byte offset of the prepared rows' stages
    static_assert(kB + NSB * B_STAGE <= 163840, "LDS budget");
    static_assert((kAStages - 1) * NI_A + (NSB - 1) * NI_B <= 63, "vmcnt range");
    __shared__ __attribute__((aligned(16))) unsigned char smem[kB + NSB * B_STAGE];
    const f32x4 *smem_a = reinterpret_cast<const f32x4 *>(smem);
    const bf16x8 *smem_b = reinterpret_cast<const bf16x8 *>(smem + kB);

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 1, wn = (w ^ (w >> 2)) & 1;     // (waves w and w + 4 share a SIMD: one of each kind)
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_void_ptr)smem;
    const int nk = p.nk;

    // ranges of the flattened (row tile, column tile, k-step) space; the projection: of (row tile, k-step), a range for
    // the n_tiles workgroups of a group, one per column tile (block id modulo 8: the XCD)
    const int across = SPLIT ? p.n_tiles : 1;
    // (an XCD's workgroups beyond its groups form groups across the XCDs)
    const int xcd = (int)blockIdx.x & 7, place = (int)blockIdx.x >> 3, left = place - p.groups * p.n_tiles;
    const int member = left < 0 ? place : left * 8 + xcd;   // of the XCD's groups, or of the others
    const int range = SPLIT ? (int)blockIdx.x : (left < 0 ? xcd : 8) * p.groups + member / p.n_tiles;
    const int64_t total = (int64_t)p.m_tiles * across * nk;
    const int64_t g_begin = (int64_t)range * p.len;
    const int64_t g_end = g_begin + p.len < total ? g_begin + p.len : total;
    if (g_begin >= g_end) return;   // uniform

    // fp32 rows: lane's place in a load instruction.  The LDS image of a row is its eight 16-byte chunks, chunk c at
    // position c ^ a_swizzle(row): a fragment read takes one chunk of each of 16 rows for every two lanes groups, and the
    // 16 lanes a cycle serves (rows 0-3 and 12-15 of one group with rows 4-11 of the next) meet 16 different positions.
    const uint32_t d4 = (uint32_t)p.d * 4;
    const uint32_t a_row = VEC ? w * WR + (lane >> 3) : w * WR + (lane >> 5);   // + i * (8 or 2)
    const uint32_t a_row_off = a_row * d4;
    // fragment addresses, in 16-byte units
    const int rA = wm * 16 * RB + (lane & 15);          // + 16 i: leaves the swizzle as it is
    const int swA = a_swizzle(rA);
    const int rdA0 = rA * 8 + ((2 * (lane >> 4)) ^ swA), rdA1 = rA * 8 + ((2 * (lane >> 4) + 1) ^ swA);
    const int rB = wn * TNB * 16 + (lane & 15);
    const int rdB = rB * 4 + ((lane >> 4) ^ tiled_chunk_swizzle(rB));

    for (int64_t g = g_begin; g < g_end;) {
        const int64_t tile = g / nk;
        const int ka = (int)(g - tile * nk);
        const int kb = g_end - tile * nk < nk ? (int)(g_end - tile * nk) : nk;
        const int nt = SPLIT ? (int)(tile % p.n_tiles) : member % p.n_tiles;
        const int64_t mt = tile / across;
        // slot: how many ranges before this one touch the tile
        const int slot = (int)(range - (tile * nk) / p.len);
        // the last row tile reaches back: every load is of a row that exists
        const int64_t row0 = (mt + 1) * ROWS <= p.n ? mt * ROWS : p.n - ROWS;
        const uint64_t gA = uniform_u64((uint64_t)(uintptr_t)(p.x + row0 * p.d));

        // load l of k-step kt's prepared rows
        auto issue_b = [&](int buf, int kt, int l) {
            int id = l * 8 + w;
            id = id < NBI ? id : NBI - 1;
            const int rb = nt * NCB + id % NCB;   // block of 16 prepared rows
            const uint64_t src = (uint64_t)(uintptr_t)(id < NCB ? p.hi : p.lo) +
                                 ((uint64_t)(rb >> 4) * (p.d_pad / kKB) + kt) * (kTileN * 64) + (rb & 15) * 1024;   // (!SPLIT: id < NCB)
            load16_global_to_lds(uniform_u64(src), lane * 16, smem_base + kB + buf * B_STAGE + id * 1024);
        };
        // load i of k-step kt's fp32 rows; elements past the row's end are met by zeros in the prepared rows: any
        // element of the row will do for them
        auto issue_a = [&](int stage, int kt, int i) {
            const uint32_t ko = (uint32_t)kt * 128;
            if constexpr (VEC) {
                const uint32_t c = (lane & 7) ^ a_swizzle(w * WR + i * 8 + (lane >> 3));
                const uint32_t at = ko + c * 16;
                const uint64_t base = gA + (uint64_t)(i * 8) * d4;
                const uint32_t off = a_row_off + (at < d4 ? at : 0u), to = smem_base + stage * kAStage + w * (WR * 128) + i * 1024;
                if constexpr (SPLIT) load16_global_to_lds_nt(base, off, to);
                else load16_global_to_lds(base, off, to);   // (the group's other workgroups ask for it too: 3,000 x 8,192 -> 700 81 us, 72 so)
            } else {
                const uint32_t at = ko + (((lane & 31) ^ (a_swizzle(w * WR + i * 2) << 2)) << 2);
                load4_global_to_lds(gA + (uint64_t)(i * 2) * d4, a_row_off + (at < d4 ? at : 0u), smem_base + stage * kAStage + w * (WR * 128) + i * 256);
            }
        };

        bf16x8 ah[2][RB], al[SPLIT ? 2 : 1][RB], bh[RING], bl[SPLIT ? 2 : 1];
        float sq[4] = {0.f, 0.f, 0.f, 0.f};
        const int tail = (int)(p.d - (int64_t)(nk - 1) * kKB);   // elements of a row's last k-step
        f32x4 raw[2];
        auto read_a = [&](int stage, int i) {
            raw[0] = smem_a[stage * (kAStage / 16) + rdA0 + i * 128];
            raw[1] = smem_a[stage * (kAStage / 16) + rdA1 + i * 128];
        };
        auto convert = [&](int set, int i, bool cut) {
            f32x8 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = raw[0][e];
                x[4 + e] = raw[1][e];
            }
            if constexpr (!SPLIT) {
                if (cut) {   // uniform: what was read past the row's end is no zero, and may be no number
                    int left = tail - (lane >> 4) * 8;
                    asm volatile("" : "+v"(left));   // (formed here: eight masks kept over the loop would spill)
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = e < left ? x[e] : 0.f;
                }
                u32x4 v = __builtin_bit_cast(u32x4, __builtin_convertvector(x, bf16x8));   // round to nearest even
                asm volatile("" : "+v"(v));   // (as below)
                ah[set][i] = __builtin_bit_cast(bf16x8, v);
                return;
            } else {
            const u32x4 h = __builtin_bit_cast(u32x4, __builtin_convertvector(x, bf16x8));   // round to nearest even
            f32x8 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                r[2 * e] = x[2 * e] - __uint_as_float(h[e] << 16);
                r[2 * e + 1] = x[2 * e + 1] - __uint_as_float(h[e] & 0xffff0000u);
            }
            u32x4 hv = h, lv = __builtin_bit_cast(u32x4, __builtin_convertvector(r, bf16x8));
            // here, among the matrix instructions, and not where the values are first used
            asm volatile("" : "+v"(hv), "+v"(lv));
            ah[set][i] = __builtin_bit_cast(bf16x8, hv);
            al[set][i] = __builtin_bit_cast(bf16x8, lv);
#pragma unroll
            for (int e = 0; e < 8; ++e) sq[i] = __builtin_fmaf(x[e], x[e], sq[i]);
            }
        };
        auto read_b = [&](int set, int buf, int j) {
            const int at = (NCB % 2 && j == TNB - 1) ? j - wn : j;   // (the second wave has no such block)
            bh[set] = smem_b[buf * (B_STAGE / 16) + rdB + at * 64];
            if constexpr (SPLIT) bl[set] = smem_b[buf * (B_STAGE / 16) + B_IMG / 16 + rdB + at * 64];
        };

        f32x4 acc[RB][TNB];
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

        const int klast = kb - 1;
        auto at_most = [&](int kt) { return kt < klast ? kt : klast; };
        __syncthreads();   // the LDS is free (a range's previous tile)
#pragma unroll
        for (int i = 0; i < NI_A; ++i) issue_a(0, ka, i);
#pragma unroll
        for (int i = 0; i < NI_A; ++i) issue_a(1, at_most(ka + 1), i);
#pragma unroll
        for (int l = 0; l < (SPLIT ? 1 : 2) * NI_B; ++l) issue_b(l / NI_B, at_most(ka + l / NI_B), l % NI_B);
#pragma unroll
        for (int i = 0; i < NI_A; ++i) issue_a(2, at_most(ka + 2), i);
        if constexpr (kAStages == 4) {
#pragma unroll
            for (int l = 0; l < NI_B; ++l) issue_b(2, at_most(ka + 2), l);
#pragma unroll
            for (int i = 0; i < NI_A; ++i) issue_a(3, at_most(ka + 3), i);
        }
        wait_global_loads_le<(kAStages - 1) * NI_A + (NSB - 1) * NI_B>();
        __syncthreads();
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            read_a(0, i);
            convert(0, i, ka == nk - 1 && tail < kKB);
        }
        wait_global_loads_le<AHEAD>();
        __syncthreads();
        int st = 0;   // stage of the fp32 rows of k-step kt
#pragma unroll
        for (int j = 0; j < PD; ++j) read_b(j, 0, j);
        // At the top of k-step kt: its A fragments are in register set `cur`, the B fragments of its first PD groups on their
        // way to registers; its prepared rows and the fp32 rows of kt + 1 are in LDS, the fp32 rows of kt + 2 in flight.  The
        // step's barrier comes before its last PD groups of matrix instructions, which need nothing newer: it publishes
        // the prepared rows of kt + 1 and the fp32 rows of kt + 2 and frees the stages of kt's prepared rows and of the fp32
        // rows of kt + 1, which have been converted.  (The projection's loads are further ahead: AHEAD.)
        auto k_step = [&](int kt, auto tag) {
            constexpr int cur = decltype(tag)::value;
            constexpr int S0 = cur * TNB;   // B fragments take RING register sets in turn, on from step to step
            const bool cut = kt + 1 == nk - 1 && tail < kKB;
            const int nst = st + 1 == kAStages ? 0 : st + 1;
            const int b_kt = at_most(kt + NSB - 1), a_kt = at_most(kt + kAStages);
            static_assert(SPLIT || NSB == kAStages, "one stage index for both");
            const int b_st = SPLIT ? cur : st, b_next = SPLIT ? cur ^ 1 : nst, b_fill = SPLIT ? cur ^ 1 : (st == 0 ? NSB - 1 : st - 1);
#pragma unroll
            for (int j = 0; j < TNB; ++j) {
                constexpr int GA = TNB - PD;   // groups that convert A blocks and issue loads
                auto group_of = [](int i) { return GA >= RB ? i : i * GA / RB; };
                auto mfma = [&](const bf16x8 &b, bf16x8(&x)[RB]) {
                    if (NCB % 2 && j == TNB - 1 && wn) return;   // uniform
#pragma unroll
                    for (int i = 0; i < RB; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, x[i], acc[i][j], 0, 0, 0);
                };
                if (j == TNB - PD) {
                    wait_global_loads_le<AHEAD>();
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    __syncthreads();
                }
                if (j + PD < TNB) {
                    read_b((S0 + j + PD) % RING, b_st, j + PD);
                    if (GA >= RB && j < RB) read_a(nst, j);
                } else {
                    read_b((S0 + j + PD) % RING, b_next, j + PD - TNB);
                }
                __builtin_amdgcn_sched_barrier(0);
                mfma(bh[(S0 + j) % RING], ah[cur]);
                if constexpr (SPLIT) mfma(bl[(S0 + j) % RING], ah[cur]);
                if (j < GA) {
#pragma unroll
                    for (int l = j * NL / GA; l < (j + 1) * NL / GA; ++l) {
                        if (l < NI_B) issue_b(b_fill, b_kt, l);
                        else issue_a(st, a_kt, l - NI_B);
                    }
                }
                if constexpr (SPLIT) mfma(bh[(S0 + j) % RING], al[cur]);
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    if (j >= GA || group_of(i) != j) continue;
                    if (GA < RB) read_a(nst, i);
                    convert(cur ^ 1, i, cut);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            st = nst;
        };
        int kt = ka;
        while (true) {
            k_step(kt, std::integral_constant<int, 0>{});
            if (++kt >= kb) break;
            k_step(kt, std::integral_constant<int, 1>{});
            if (++kt >= kb) break;
        }
        wait_global_loads_le<0>();   // the refills past the last k-step
        // Sums out: the matrix instruction takes the prepared rows as its rows, so a lane holds four consecutive
        // columns of one fp32 row.
        if constexpr (!SPLIT) {
            if (ka == 0 && kb == nk) {   // uniform: the whole tile.  (Rows that the last row tile reaches back over are the one's before it.)
#pragma unroll
                for (int i = 0; i < RB; ++i) {
                    const int64_t row = row0 + wm * 16 * RB + i * 16 + (lane & 15);
                    if (row < mt * ROWS) continue;
#pragma unroll
                    for (int j = 0; j < TNB; ++j) store_projected(p, row, nt * NC + (wn * TNB + j) * 16 + (lane >> 4) * 4, acc[i][j]);
                }
                g = tile * nk + kb;
                continue;
            }
        }
        float *dst = p.part + (((SPLIT ? tile : mt * p.n_tiles + nt) * p.slots + slot) * ROWS + wm * 16 * RB + (lane & 15)) * NC + wn * TNB * 16 + (lane >> 4) * 4;
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
                if (wn * TNB + j < NCB) *reinterpret_cast<f32x4 *>(dst + i * 16 * NC + j * 16) = acc[i][j];
        if (SPLIT && nt == 0 && wn == 0) {
            // (the fragments converted past the last k-step are of that step again: sums of squares only grow by them; and by what
            // stands in for the elements past the row's end, which the reader takes off)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float v = sq[i];
                v += __shfl_xor(v, 16, 64);
                v += __shfl_xor(v, 32, 64);
                if (lane < 16) p.sq[(mt * p.slots + slot) * kRowsTile + wm * 64 + i * 16 + lane] = v;
            }
        }
        g = tile * nk + kb;
    }
}

// The projection's output where ranges cut its tiles: the sums of a tile's slots, in order, kSumRows rows of a tile per
// workgroup.
constexpr int kSumRows = 4;
__global__ __launch_bounds__(256) void project_sum_kernel(RowsGemmArgs p, int nc)
{
    const int rows = p.rows;   // of a tile
    const int64_t tile = blockIdx.x / (rows / kSumRows), mt = tile / p.n_tiles;
    const int64_t first = mt * p.nk / p.len, last = (mt * p.nk + p.nk - 1) / p.len;
    if (first == last) return;   // uniform: written by its range
    const int ns = (int)(last - first) + 1, nt = (int)(tile - mt * p.n_tiles);
    const int64_t row0 = (mt + 1) * rows <= p.n ? mt * rows : p.n - rows;
    const int r0 = (int)(blockIdx.x % (rows / kSumRows)) * kSumRows, q = nc / 4;
    for (int i = threadIdx.x; i < kSumRows * q; i += 256) {
        const int r = r0 + i / q, c = i % q * 4;
        if (row0 + r < mt * rows || (int64_t)nt * nc + c >= p.m) continue;
        const float *src = p.part + (tile * p.slots * rows + r) * nc + c;
        const int64_t step = (int64_t)rows * nc;
        // four in flight, and four summed before they are added: one after the other, the error of sums of 40 slots was a quarter larger
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < ns; s += 4) {
            f32x4 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                t[u] = *reinterpret_cast<const f32x4 *>(src + (s + u < ns ? s + u : s) * step);
                if (s + u >= ns) t[u] = f32x4{0.f, 0.f, 0.f, 0.f};   // uniform
            }
            v += (t[0] + t[1]) + (t[2] + t[3]);
        }
        store_projected(p, row0 + r, (int64_t)nt * nc + c, v);
    }
}

// hi, lo [tile of kTileN rows][k-block][row][32] and norm of the fp32 rows [kc, d]: x = hi + lo up to 2^-17 |x|.  Rows past
// kc are zeros with norm +inf.
__global__ __launch_bounds__(512) void rows_split_kernel(const float *rows, int64_t kc, int64_t d, int64_t d_pad, uint16_t *hi, uint16_t *lo, float *norm)
{
    __shared__ double wave_sum[8];
    const int64_t r = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t base = (r / kTileN) * (int64_t)kTileN * d_pad;
    double s = 0.0;
    for (int64_t j = tid; j < d_pad / 8; j += 512) {
        __attribute__((aligned(16))) uint16_t h[8], l[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t at = j * 8 + e;
            const float x = r < kc && at < d ? rows[r * d + at] : 0.f;
            h[e] = bf16_rne(x);
            l[e] = bf16_rne(x - __uint_as_float((uint32_t)h[e] << 16));
            s += (double)x * (double)x;
        }
        const int64_t o = base + tiled_chunk_offset((int)(r % kTileN), j, kTileN) * 8;
        *reinterpret_cast<uint4 *>(hi + o) = *reinterpret_cast<const uint4 *>(h);
        *reinterpret_cast<uint4 *>(lo + o) = *reinterpret_cast<const uint4 *>(l);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) wave_sum[w] = s;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int i = 0; i < 8; ++i) t += wave_sum[i];
        norm[r] = r < kc ? (float)t : __builtin_inff();
    }
}

struct PickArgs {
    const float *x, *centers;   // [n, d], [kc, d]
    const float *part, *sq, *norm;
    int32_t *assign;
    int64_t n, d, kc;
    uint32_t len;               // (the flattened space has fewer than 2^31 k-steps)
    int nk, n_tiles, slots, nc;
    float eps;                  // bound of a key's error, in units of 2 |q||c| (key_error)
    bool wide;                  // wide_order(n, d)
};

constexpr int kPickPoints = 4;   // points per wave

// fp32 distances of point row q to the m centres cand_s, by 256 threads, in the order of additions that the look-ups'
// re-scoring has for rows of this length (rescore_block_all<256, .> and rescore_wave; wide: rescore_block_all<1024, .>, four
// threads' chains by each): whoever assigns a point, nearly equal distances compare alike.
__device__ inline void exact_distances(const float *q, const float *centers, int64_t d, bool wide, const int32_t *cand_s, int m, float *dist_s, float *red_s, int tid)
{
    const int lane = tid & 63, w = tid >> 6;
    auto wave_sum = [](float v) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        return v;
    };
    auto eight = [](const f32x4 (&x)[2], const f32x4 (&c)[2], float acc) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float df = x[e >> 2][e & 3] - c[e >> 2][e & 3];
            acc = __builtin_fmaf(df, df, acc);
        }
        return acc;
    };
    // chain of pieces of eight elements at first, first + step, .., four pieces' loads in flight
    auto chain = [&](const float *r, int64_t first, int64_t step) {
        float acc = 0.f;
        int64_t i = first;
        for (; i + 3 * step < d; i += 4 * step) {
            f32x4 x[4][2], c[4][2];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    x[u][h] = *reinterpret_cast<const f32x4 *>(q + i + u * step + 4 * h);
                    c[u][h] = *reinterpret_cast<const f32x4 *>(r + i + u * step + 4 * h);
                }
#pragma unroll
            for (int u = 0; u < 4; ++u) acc = eight(x[u], c[u], acc);
        }
        for (; i < d; i += step) {
            const f32x4 x[2] = {*reinterpret_cast<const f32x4 *>(q + i), *reinterpret_cast<const f32x4 *>(q + i + 4)};
            const f32x4 c[2] = {*reinterpret_cast<const f32x4 *>(r + i), *reinterpret_cast<const f32x4 *>(r + i + 4)};
            acc = eight(x, c, acc);
        }
        return acc;
    };
    if (d >= 4096 && d % 8 == 0) {   // (rows start on 16-byte boundaries)
        const int parts = wide ? 4 : 1;
        for (int j = 0; j < m; ++j) {
            float t = 0.f;
            for (int part = 0; part < parts; ++part) {
                const float v = wave_sum(chain(centers + cand_s[j] * d, (int64_t)(part * 256 + tid) * 8, parts * 256 * 8));
                if (lane == 0) red_s[w] = v;
                __syncthreads();
                t += (red_s[0] + red_s[1]) + (red_s[2] + red_s[3]);
                __syncthreads();
            }
            if (tid == 0) dist_s[j] = t;
        }
        __syncthreads();
        return;
    }
    for (int j = w; j < m; j += 4) {
        const float *r = centers + cand_s[j] * d;
        float acc = 0.f;
        if (d % 8 == 0) {
            acc = chain(r, (int64_t)lane * 8, 64 * 8);
        } else {
            int64_t i = lane;
            for (; i + 3 * 64 < d; i += 4 * 64) {
                float x[4], c[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    x[u] = q[i + u * 64];
                    c[u] = r[i + u * 64];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float df = x[u] - c[u];
                    acc = __builtin_fmaf(df, df, acc);
                }
            }
            for (; i < d; i += 64) {
                const float df = q[i] - r[i];
                acc = __builtin_fmaf(df, df, acc);
            }
        }
        acc = wave_sum(acc);
        if (lane == 0) dist_s[j] = acc;
    }
    __syncthreads();
}

// Nearest centre of every point, kPickPoints points per wave.  key(c) = |c|^2 - 2 q.c is off by at most
//     e(c) = 2 eps |q||c| + 2^-22 (|c|^2 + |q|^2),  eps = key_error():
// the second term covers the rounding of |c|^2 and of the last subtraction.  Centres with key - e above the smallest key + e
// are not the nearest.  If more than one is left, the workgroup re-scores them exactly; equal distances go to the lower index.
// Keys that are no numbers (overflow) leave all centres in.
template <int MT>   // centre tiles
__global__ __launch_bounds__(256) void kmeans_pick_kernel(PickArgs p)
{
    constexpr int U = kPickPoints;
    const int lane = threadIdx.x & 63;
    const int64_t i0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * U;   // (U divides kRowsTile: one row tile)
    // (a wave past the end goes through the motions on the last point: the workgroup's barriers need it)
    const int live = i0 >= p.n ? 0 : (p.n - i0 < U ? (int)(p.n - i0) : U);
    const int64_t at0 = live ? i0 : p.n - 1;
    const int64_t m_tile = at0 / kRowsTile;
    const int64_t row0 = (m_tile + 1) * kRowsTile <= p.n ? m_tile * kRowsTile : p.n - kRowsTile;
    const int row = (int)(at0 - row0);
    auto slots_of = [&](int64_t tile) {
        const uint32_t at = (uint32_t)tile * (uint32_t)p.nk;
        return p.slots == 1 ? 1 : (int)((at + p.nk - 1) / p.len - at / p.len) + 1;
    };
    float q2[U];
#pragma unroll
    for (int u = 0; u < U; ++u) q2[u] = 0.f;
    {
        const int ns = slots_of(m_tile * p.n_tiles);
        for (int s = 0; s < ns; ++s)
#pragma unroll
            for (int u = 0; u < U; ++u)
                q2[u] += p.sq[(m_tile * p.slots + s) * kRowsTile + row + (u < live ? u : 0)];
        // What stood in for the elements past the row's end in its last k-step (converted twice): the row's first four values for
        // every four of them, or its first value for each.  Taken off again, less the rounding of the sum: a large first
        // channel would widen the bound (50,000 x 8,200, 200 centres, the first value a hundred times the others: 2,950 us,
        // now 2,570; 8,199 values 3,700, 2,510).
        const int past = p.nk * kKB - (int)p.d;
        if (past > 0) {   // uniform
            const int values = p.d % 4 == 0 ? 4 : 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float *x = p.x + (at0 + (u < live ? u : 0)) * p.d;
                float first = 0.f;
                for (int e = 0; e < values; ++e) first = __builtin_fmaf(x[e], x[e], first);
                q2[u] = __builtin_fmaxf(q2[u] - (float)(2 * past / values) * first, 0.f) + 5.97e-8f * (8.f * (float)p.nk + 64.f) * q2[u];
            }
        }
    }
    // columns of a lane: 4 lane .. + 3 of every column tile (a tile has at most 256)
    float lower[U][MT][4], upper[U];
#pragma unroll
    for (int u = 0; u < U; ++u) upper[u] = __builtin_inff();
#pragma unroll
    for (int t = 0; t < MT; ++t) {
        if (t >= p.n_tiles || 4 * lane >= p.nc) continue;
        const int64_t tile = m_tile * p.n_tiles + t;
        const int ns = slots_of(tile);
        const float *src = p.part + (tile * p.slots * kRowsTile + row) * p.nc + 4 * lane;
        f32x4 dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) dot[u] = *reinterpret_cast<const f32x4 *>(src + (u < live ? u : 0) * p.nc);
        for (int s = 1; s < ns; ++s)
#pragma unroll
            for (int u = 0; u < U; ++u) dot[u] += *reinterpret_cast<const f32x4 *>(src + ((int64_t)s * kRowsTile + (u < live ? u : 0)) * p.nc);
        // (the norms' buffer has whole tiles of kTileN entries, +inf past the last centre)
        const f32x4 c2 = *reinterpret_cast<const f32x4 *>(p.norm + t * p.nc + 4 * lane);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float c1 = __builtin_sqrtf(c2[e]);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float key = __builtin_fmaf(-2.f, dot[u][e], c2[e]);
                const float err = 2.f * p.eps * __builtin_sqrtf(q2[u]) * c1 + 2.4e-7f * (c2[e] + q2[u]) + 1e-36f * (float)p.d;
                lower[u][t][e] = key - err;
                if ((int64_t)t * p.nc + 4 * lane + e < p.kc) upper[u] = __builtin_fminf(upper[u], key + err);
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
        for (int u = 0; u < U; ++u) upper[u] = __builtin_fminf(upper[u], __shfl_xor(upper[u], off, 64));
    // masks[point][lane]: the lane's centres that are left (bit 4 t + e: column 4 lane + e of tile t), where more than one is
    __shared__ uint32_t masks[4 * U][64];
    __shared__ int open_s[4 * U];
    __shared__ int32_t cand_s[MT * 256];
    __shared__ float dist_s[MT * 256];
    __shared__ float red_s[4];
    __shared__ int count_s;
    const int w = threadIdx.x >> 6;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        uint32_t mine = 0;
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (t < p.n_tiles && 4 * lane < p.nc && (int64_t)t * p.nc + 4 * lane + e < p.kc && !(lower[u][t][e] > upper[u])) mine |= 1u << (t * 4 + e);
        const uint64_t any = __ballot(mine != 0);
        const uint32_t only = (uint32_t)__builtin_amdgcn_readlane((int)mine, any ? __builtin_ctzll(any) : 0);
        const bool one = any && (any & (any - 1)) == 0 && (only & (only - 1)) == 0;
        masks[w * U + u][lane] = mine;
        if (lane == 0) {
            open_s[w * U + u] = u < live && !one;
            const int bit = __builtin_ctz(only | 0x80000000u);
            if (u < live && one) p.assign[i0 + u] = (int32_t)((bit >> 2) * p.nc + 4 * __builtin_ctzll(any) + (bit & 3));
        }
    }
    __syncthreads();
    for (int o = 0; o < 4 * U; ++o) {
        if (!open_s[o]) continue;   // uniform
        const int64_t i = (int64_t)blockIdx.x * 4 * U + o;
        if (w == 0) {   // the centres that are left, ascending
            const uint32_t mine = masks[o][lane];
            int base = 0;
            for (int t = 0; t < p.n_tiles; ++t) {
                const uint32_t bits = mine >> (t * 4) & 15u;
                const int own = __builtin_popcount(bits);
                int at = own;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const int v = __shfl_up(at, off, 64);
                    if (lane >= off) at += v;
                }
                const int all = __shfl(at, 63, 64);
                at += base - own;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (bits >> e & 1u) cand_s[at++] = t * p.nc + 4 * lane + e;
                base += all;
            }
            if (lane == 0) count_s = base;
        }
        __syncthreads();
        const int m = count_s;
        exact_distances(p.x + i * p.d, p.centers, p.d, p.wide, cand_s, m, dist_s, red_s, (int)threadIdx.x);
        if (w == 0) {   // the nearest, equal distances the lower index (which comes first)
            uint64_t best = kSentinel;
            for (int j = lane; j < m; j += 64) {
                const uint64_t v = ((uint64_t)ordered_bits(dist_s[j]) << 32) | (uint32_t)j;
                best = v < best ? v : best;
            }
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const uint64_t v = ((uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(best >> 32), off, 64) << 32) | (uint32_t)__shfl_xor((int)(uint32_t)best, off, 64);
                best = v < best ? v : best;
            }
            const uint32_t j = (uint32_t)best;
            if (lane == 0) p.assign[i] = cand_s[j < (uint32_t)m ? j : 0];
        }
        __syncthreads();   // cand_s and dist_s are free
    }
}

template <int NCB, bool SPLIT, int RB = 4>
hipError_t launch_gemm(const RowsPlan &pl, const RowsGemmArgs &a, hipStream_t s)
{
    if (a.d % 4 == 0)
        hipLaunchKernelGGL((rows_gemm_kernel<NCB, true, SPLIT, RB>), dim3((unsigned)pl.wgs), dim3(512), 0, s, a);
    else
        hipLaunchKernelGGL((rows_gemm_kernel<NCB, false, SPLIT, RB>), dim3((unsigned)pl.wgs), dim3(512), 0, s, a);
    return hipGetLastError();
}

}  // namespace

RowsPlan plan_rows(int64_t n, int64_t d, int64_t kc, int num_cus)
{
    RowsPlan pl{};
    // a tile's rows reach 4 GiB at most; the last row tile reaches back over the one before it
    if (n < kRowsTile || d < 1 || d > (int64_t)1 << 20 || kc < 1 || kc > kRowsMaxTiles * kTileN) return pl;
    pl.n_tiles = (int)((kc + kTileN - 1) / kTileN);
    const int per = (int)((kc + pl.n_tiles - 1) / pl.n_tiles);
    // As many blocks of columns as are needed, four at least.  An odd number's waves differ, which costs registers and still is 1
    // to 5 % of a build less than the next even one (50,000 x 8,192 with 136 centres 1,937 -> 1,880 us, 168 2,068 -> 2,010, 200
    // 2,230 -> 2,151, 280 3,156 -> 3,043; 9,000 x 1,023 with 104 250 -> 242); of 15 blocks 18 registers spill: 50,000 x 8,192
    // with 232 2,312 -> 2,264, but 20,000 x 4,100 with 480 1,320 -> 1,332, 50,000 x 517 with 232 524 -> 536.
    pl.ncb = per <= 64 ? 4 : (per + 15) / 16;
    if (pl.ncb == 15) pl.ncb = 16;
    pl.nc = 16 * pl.ncb;
    pl.m_tiles = (int)((n + kRowsTile - 1) / kRowsTile);
    pl.nk = (int)((d + kKB - 1) / kKB);
    const int64_t tiles = (int64_t)pl.m_tiles * pl.n_tiles, total = tiles * pl.nk;
    if (tiles >= 8 * (int64_t)num_cus) {
        pl.len = (tiles + num_cus - 1) / num_cus * pl.nk;   // whole tiles: an idle eighth at most
    } else {
        pl.len = (total + num_cus - 1) / num_cus;
        const int64_t least = pl.nk < 8 ? pl.nk : 8;        // a slot is written and read for it
        if (pl.len < least) pl.len = least;
    }
    pl.wgs = (int)((total + pl.len - 1) / pl.len);
    pl.slots = pl.len % pl.nk == 0 ? 1 : (int)((pl.nk + pl.len - 2) / pl.len) + 1;
    pl.part = (size_t)tiles * pl.slots * kRowsTile * pl.nc;
    pl.sq = (size_t)pl.m_tiles * pl.slots * kRowsTile;
    pl.on = pl.part * 4 <= (size_t)1 << 30 && total < (int64_t)1 << 31;
    return pl;
}

// Bound of |q.c - what the product makes of it| / (|q||c|).
//   - lo.lo, at most 2^-16 of |q||c|, and what hi + lo leaves of the values, 2^-17 of each: 2^-15 and a little.
//   - Additions.  A matrix instruction takes its 32 products in four groups of eight (measured on single bits): a group's products
//     are summed with what lies under 2^-24 of the largest cut off, and the accumulator takes each sum with one rounding to
//     nearest.  Three instructions per k-step: twelve roundings, each 2^-24 of a partial sum at most, and partial sums are
//     at most |q||c|.  They all go the same way where the addends are alike (rows of nearly constant values: with
//     sqrt(3 nk) 2^-24 times eight, as if they were independent, 408 of 512 clusters of 32,768 constant rows of
//     65,536 values took points of others), so their number counts and not its root.  Sums that a range's end cuts begin anew; then
//     one more addition per slot.  The cut-off parts come to 8 2^-24 of all products.
//   - |q| comes from 8 nk additions of squares.
static float key_error(const RowsPlan &pl)
{
    const float chain = (float)(pl.len < pl.nk ? pl.len : pl.nk);
    return (3.1e-5f + 5.97e-8f * (12.f * chain + (float)pl.slots + 12.f)) * (1.f + 5.97e-8f * 8.f * (float)pl.nk);
}

hipError_t launch_rows_split(const float *rows, int64_t kc, int64_t n_pad, int64_t d, int64_t d_pad, uint16_t *hi, uint16_t *lo, float *norm, hipStream_t s)
{
    hipLaunchKernelGGL(rows_split_kernel, dim3((unsigned)n_pad), dim3(512), 0, s, rows, kc, d, d_pad, hi, lo, norm);
    return hipGetLastError();
}

hipError_t launch_kmeans_assign(const RowsPlan &pl, const float *points, int64_t n, int64_t d, int64_t d_pad, const float *centers, int64_t kc,
                                const uint16_t *hi, const uint16_t *lo, const float *norm, float *part, float *sq, int32_t *assign, hipStream_t s)
{
    if (!pl.on || n < kRowsTile || pl.m_tiles != (n + kRowsTile - 1) / kRowsTile || d_pad < (int64_t)pl.nk * kKB || kc > (int64_t)pl.n_tiles * pl.nc ||
        (int64_t)pl.n_tiles * pl.nc > (kc + kTileN - 1) / kTileN * kTileN || (reinterpret_cast<uintptr_t>(points) % 16) != 0)
        return hipErrorInvalidValue;
    RowsGemmArgs a{points, hi, lo, part, sq, n, d, d_pad, pl.len, pl.nk, pl.n_tiles, pl.m_tiles, pl.slots, kRowsTile, 0, nullptr, nullptr, 0, 0};
    hipError_t e;
    switch (pl.ncb) {
    case 4: e = launch_gemm<4, true>(pl, a, s); break;
    case 5: e = launch_gemm<5, true>(pl, a, s); break;
    case 6: e = launch_gemm<6, true>(pl, a, s); break;
    case 7: e = launch_gemm<7, true>(pl, a, s); break;
    case 8: e = launch_gemm<8, true>(pl, a, s); break;
    case 9: e = launch_gemm<9, true>(pl, a, s); break;
    case 10: e = launch_gemm<10, true>(pl, a, s); break;
    case 11: e = launch_gemm<11, true>(pl, a, s); break;
    case 12: e = launch_gemm<12, true>(pl, a, s); break;
    case 13: e = launch_gemm<13, true>(pl, a, s); break;
    case 14: e = launch_gemm<14, true>(pl, a, s); break;
    case 16: e = launch_gemm<16, true>(pl, a, s); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    PickArgs k{points, centers, part, sq, norm, assign, n, d, kc, (uint32_t)pl.len, pl.nk, pl.n_tiles, pl.slots, pl.nc, key_error(pl), wide_order(n, d)};
    const dim3 grid((unsigned)((n + 4 * kPickPoints - 1) / (4 * kPickPoints)));
    if (pl.n_tiles == 1) hipLaunchKernelGGL(kmeans_pick_kernel<1>, grid, dim3(256), 0, s, k);
    else hipLaunchKernelGGL(kmeans_pick_kernel<kRowsMaxTiles>, grid, dim3(256), 0, s, k);
    return hipGetLastError();
}

// across: with the workgroups beyond the groups of their XCD, in groups across the XCDs
static RowsPlan plan_projection_rows(int64_t n, int64_t d, int64_t m, int num_cus, int rows, bool across)
{
    RowsPlan pl{};
    pl.rows = rows;
    const int per_xcd = num_cus / 8;
    if (n < rows || d < 1 || d > (int64_t)1 << 20 || m < 1 || m > (int64_t)per_xcd * kTileN) return pl;
    pl.n_tiles = (int)((m + kTileN - 1) / kTileN);
    const int per = (int)((m + pl.n_tiles - 1) / pl.n_tiles);
    pl.ncb = per <= 128 ? 8 : (per <= 192 ? 12 : 16);
    pl.nc = 16 * pl.ncb;
    pl.m_tiles = (int)((n + rows - 1) / rows);
    pl.nk = (int)((d + kKB - 1) / kKB);
    pl.groups = per_xcd / pl.n_tiles;
    const int64_t total = (int64_t)pl.m_tiles * pl.nk;
    auto range_len = [&](int64_t ranges) {
        if (pl.m_tiles >= 8 * ranges) return (pl.m_tiles + ranges - 1) / ranges * pl.nk;   // whole tiles: an idle eighth at most
        const int64_t len = (total + ranges - 1) / ranges, least = pl.nk < 8 ? pl.nk : 8;   // a slot is written and read for it
        return len < least ? least : len;
    };
    pl.len = range_len(8 * pl.groups);
    // (not where ranges are whole tiles without them)
    if (across && pl.len % pl.nk != 0) pl.len = range_len(8 * pl.groups + 8 * (per_xcd - pl.groups * pl.n_tiles) / pl.n_tiles);
    pl.wgs = 8 * per_xcd;   // (ranges past the end return at once)
    pl.slots = pl.len % pl.nk == 0 ? 1 : (int)((pl.nk + pl.len - 2) / pl.len) + 1;
    pl.part = pl.slots == 1 ? 0 : (size_t)pl.m_tiles * pl.n_tiles * pl.slots * rows * pl.nc;
    pl.on = pl.part * 4 <= (size_t)1 << 30;
    return pl;
}

// Tiles of 256 rows take 1.22 us a k-step, of 192 rows 0.94 where the chip is busy (10,000 x 8,192 -> 1,024: what L2
// hands to the CUs, 10 TB/s, bounds both: 210, 219 us) and about 0.8 in short ranges (1,500 x 8,192 -> 1,024, 24 and 32 k-steps: 55, 46;
// 3,000 x 8,192 -> 700 67, 60; but 2,000 x 16,384 -> 256, 16 and 22 k-steps: 53, 58).
// The length of a chain of additions is part of the projection's precision: where the faster one's is more than `most` k-steps, the
// one with shorter sums (6,079 x 8,192 -> 1,024: 129 us with an error of 3.2e-7 against 64 bits, 148 with 2.56e-7, that of
// 256 x 256 tiles dealt evenly to the CUs).
RowsPlan plan_projection(int64_t n, int64_t d, int64_t m, int num_cus, int64_t most)
{
    const RowsPlan p4 = plan_projection_rows(n, d, m, num_cus, 256, false), p3 = plan_projection_rows(n, d, m, num_cus, 192, false);
    if (!p4.on || !p3.on) return plan_projection_rows(n, d, m, num_cus, p4.on ? 256 : 192, true);
    const bool large = p3.len * 100 >= p4.len * (p4.len >= 128 || p4.slots == 1 ? 130 : 136);
    const RowsPlan fast = plan_projection_rows(n, d, m, num_cus, large ? 256 : 192, true);
    if (std::min<int64_t>(fast.len, fast.nk) <= most) return fast;
    const RowsPlan other = plan_projection_rows(n, d, m, num_cus, large ? 192 : 256, true);
    return other.len < fast.len ? other : fast;
}

hipError_t launch_project(const RowsPlan &pl, const float *x, int64_t n, int64_t d, int64_t d_pad, const uint16_t *w, int64_t m, int64_t m_pad,
                          const float *bias, bool relu, float *part, float *out, hipStream_t s)
{
    if (!pl.on || (pl.rows != 192 && pl.rows != 256) || n < pl.rows || pl.m_tiles != (n + pl.rows - 1) / pl.rows || pl.nk != (d + kKB - 1) / kKB || d_pad < (int64_t)pl.nk * kKB ||
        m > (int64_t)pl.n_tiles * pl.nc || (int64_t)pl.n_tiles * pl.nc > m_pad || (pl.part > 0 && !part) ||
        ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(out)) % 16) != 0)
        return hipErrorInvalidValue;
    RowsGemmArgs a{x, w, nullptr, part, nullptr, n, d, d_pad, pl.len, pl.nk, pl.n_tiles, pl.m_tiles, pl.slots, pl.rows, pl.groups, bias, out, m, relu ? 1 : 0};
    hipError_t e;
    switch (pl.ncb) {
    case 8: e = pl.rows == 192 ? launch_gemm<8, false, 3>(pl, a, s) : launch_gemm<8, false, 4>(pl, a, s); break;
    case 12: e = pl.rows == 192 ? launch_gemm<12, false, 3>(pl, a, s) : launch_gemm<12, false, 4>(pl, a, s); break;
    case 16: e = pl.rows == 192 ? launch_gemm<16, false, 3>(pl, a, s) : launch_gemm<16, false, 4>(pl, a, s); break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess || pl.slots == 1) return e;
    hipLaunchKernelGGL(project_sum_kernel, dim3((unsigned)(pl.m_tiles * pl.n_tiles * (pl.rows / kSumRows))), dim3(256), 0, s, a, pl.nc);
    return hipGetLastError();
}

}  // namespace fz
