// Kernels around the distance pass: cache ingest, query preparation, the finishing
// kernels (merge of per-split candidate lists, exact fp32 re-scoring, final top-k, the
// certificate that no entry outside the candidates can be nearer, label vote, hit decision;
// the wider re-scoring and the exact fp32 scan for queries the certificate does not confirm;
// the one-launch finish of the small-batch path), miss compaction, the cascade's scatter, the
// row gather and the threshold calibration.  gfx950 only.
#include "freeze_internal.h"
#include "select_common.h"

#include <type_traits>

namespace fz {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
// 16-byte loads of what starts on a multiple of its element's size only (rows of odd length): the memory system takes
// them whole, where eight loads per lane of one element each fetch every line eight times over
typedef f32x4 __attribute__((aligned(4))) f32x4_any;
typedef u32x4 __attribute__((aligned(2))) u32x4_any;

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Sum over the 256 threads of a block in a fixed order; result valid in every thread.
__device__ __forceinline__ float block_sum_256(float v, float *scratch4)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) scratch4[w] = v;
    __syncthreads();
    return (scratch4[0] + scratch4[1]) + (scratch4[2] + scratch4[3]);
}

// ---------------------------------------------------------------------------------------
// Cache ingest (Pseudocode 1, ConstructCache: the layer's list of <output, label>).
// One block per padded cache row: bf16 copy (round to nearest even when given fp32) into the
// tiled layout, zero padding, |c|^2 of the bf16 row in fp32, and a row-major copy of the stored
// values for exact re-scoring (fp32 rows when the cache was given in fp32, else bf16 rows): the
// re-scoring gathers whole rows, which the tiled layout would serve in half-used cache lines.
// ---------------------------------------------------------------------------------------
// Centring of the matrix-core copy.  Distances do not change when the same vector is subtracted
// from entries and queries, but the coarse key |c|^2 - 2 q.c does: for a cache that sits far from
// the origin both of its terms are huge next to the distance and their bf16 / fp32 rounding swamps
// the differences between neighbours.  So the bf16 copy the matrix cores read (and the queries'
// bf16 copy) may be taken relative to the cache's mean vector mu; the stored values, which the exact
// re-scoring reads, stay as they are.  Whether to do so is decided on the device from the column
// statistics: only when the mean dominates the spread (|mu|^2 > 4 * total variance); otherwise mu is
// all zeros, the subtraction is exact and the copy is the plain rounding of the stored values (for
// a cache stored in bf16 centring adds a rounding error the plain copy does not have).
//
// The statistics come from a sample of at most kStatRows rows, evenly spaced over the cache (all
// rows of a smaller cache): mu may be any vector, the results never depend on it, and the
// decision needs no more precision than that.
//
// Column sums and sums of squares of the sampled rows in fp64: block (x, y) takes 512 columns (eight
// per lane, so that a wave reads 1 KiB, or 2 KiB of fp32, of a row at a time) and a range of the
// sample; its sixteen waves take every sixteenth row of that range.  What bounds it are the fp64 atomic additions that a
// workgroup ends with (two per column): few, large workgroups.
constexpr int kStatRows = 8192;
constexpr int kStatWaves = 16;
__global__ __launch_bounds__(64 * kStatWaves) void col_stats_kernel(const void *entries, int dtype, int64_t n, int64_t d, int64_t d_pad,
                                                        int64_t ns, double *stats)
{
    __shared__ double comb[kStatWaves - 1][16][64], own[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t col = ((int64_t)blockIdx.x * 64 + lane) * 8;
    const int64_t per = (ns + gridDim.y - 1) / gridDim.y;
    const int64_t i0 = (int64_t)blockIdx.y * per, i1 = i0 + per < ns ? i0 + per : ns;
    const bool vec = col + 8 <= d;
    const uint64_t step = ((uint64_t)n << 32) / (uint64_t)ns;   // ns <= 8,192, i < ns: no overflow below 2^31 rows
    double s1[8], s2[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) s1[e] = s2[e] = 0.0;
    if (col < d) {
        int64_t i = i0 + w;
        if (vec) {
            // whole groups of values, four rows in flight; sample i of ns is row i * n / ns (n / ns in 32.32 fixed
            // point: distinct rows, for ns <= n)
            constexpr int U = 4;
            for (; i + kStatWaves * (U - 1) < i1; i += kStatWaves * U) {
                f32x4 f[U][2];
                u32x4 u[U];
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    const int64_t r = (int64_t)(((uint64_t)(i + kStatWaves * t) * step) >> 32);
                    if (dtype == 0) {
                        const float *src = reinterpret_cast<const float *>(entries) + r * d + col;
                        f[t][0] = *reinterpret_cast<const f32x4_any *>(src);
                        f[t][1] = *reinterpret_cast<const f32x4_any *>(src + 4);
                    } else {
                        u[t] = *reinterpret_cast<const u32x4_any *>(reinterpret_cast<const uint16_t *>(entries) + r * d + col);
                    }
                }
#pragma unroll
                for (int t = 0; t < U; ++t) {
                    float v[8];
                    if (dtype == 0) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = f[t][e >> 2][e & 3];
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            v[2 * e] = __uint_as_float(u[t][e] << 16);
                            v[2 * e + 1] = __uint_as_float(u[t][e] & 0xffff0000u);
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        s1[e] += (double)v[e];
                        s2[e] += (double)v[e] * (double)v[e];
                    }
                }
            }
        }
        for (; i < i1; i += kStatWaves) {
            const int64_t r = (int64_t)(((uint64_t)i * step) >> 32);
            float v[8];
            if (vec && dtype == 0) {
                const float *src = reinterpret_cast<const float *>(entries) + r * d + col;
                const f32x4 v0 = *reinterpret_cast<const f32x4_any *>(src), v1 = *reinterpret_cast<const f32x4_any *>(src + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = v0[e];
                    v[4 + e] = v1[e];
                }
            } else if (vec) {
                const u32x4 wv = *reinterpret_cast<const u32x4_any *>(reinterpret_cast<const uint16_t *>(entries) + r * d + col);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] = __uint_as_float(wv[e] << 16);
                    v[2 * e + 1] = __uint_as_float(wv[e] & 0xffff0000u);
                }
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = col + e >= d ? 0.f
                                        : (dtype == 0 ? reinterpret_cast<const float *>(entries)[r * d + col + e]
                                                      : bf16_to_f32(reinterpret_cast<const uint16_t *>(entries)[r * d + col + e]));
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                s1[e] += (double)v[e];
                s2[e] += (double)v[e] * (double)v[e];
            }
        }
    }
    if (w > 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            comb[w - 1][e][lane] = s1[e];
            comb[w - 1][8 + e][lane] = s2[e];
        }
    }
    // sum t of 16 of a lane's columns by wave t: the waves' sums in order
    if (w == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            own[e][lane] = s1[e];
            own[8 + e][lane] = s2[e];
        }
    }
    __syncthreads();
    const int e = w & 7;
    if (col + e < d) {
        double t = own[w][lane];
        for (int u = 0; u < kStatWaves - 1; ++u) t += comb[u][w][lane];
        atomicAdd(&stats[(w >> 3) * d_pad + col + e], t);
    }
}

// mu[i] = column mean (or 0 everywhere when the cache is not worth centring); one workgroup
__global__ __launch_bounds__(1024) void col_mean_kernel(const double *stats, int64_t n, int64_t d, int64_t d_pad, int mode,
                                                        float *mu)
{
    __shared__ double red_m[16], red_v[16];
    __shared__ int centre_s;
    const int tid = threadIdx.x;
    double m2 = 0.0, var = 0.0;
    for (int64_t i = tid; i < d; i += 1024) {
        const double mean = stats[i] / (double)n;
        const double v = stats[d_pad + i] / (double)n - mean * mean;
        m2 += mean * mean;
        var += v > 0.0 ? v : 0.0;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        m2 += __shfl_xor(m2, off, 64);
        var += __shfl_xor(var, off, 64);
    }
    if ((tid & 63) == 0) {
        red_m[tid >> 6] = m2;
        red_v[tid >> 6] = var;
    }
    __syncthreads();
    if (tid == 0) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < 16; ++w) {
            a += red_m[w];
            b += red_v[w];
        }
        centre_s = mode == 2 || (mode == 1 && a > 4.0 * b);
    }
    __syncthreads();
    const bool centre = centre_s != 0;
    for (int64_t i = tid; i < d_pad; i += 1024) mu[i] = (centre && i < d) ? (float)(stats[i] / (double)n) : 0.f;
}

// RB rows per workgroup (16; 4 for caches of few rows, which would otherwise leave most CUs without work)
template <int RB>
__global__ __launch_bounds__(256) void cache_build_kernel(const void *entries, int dtype, int64_t n, int64_t d,
                                                          int64_t d_pad, uint16_t *c_bf, float *norm, float *c_f32,
                                                          uint16_t *c_rows, const float *mu, const int32_t *labels_in,
                                                          int32_t *labels_out)
{
    // the matrix cores' copy of the block's rows, 64 chunks (512 elements) of every row at a time, on its
    // way from row order to the tiled order (rows padded by one chunk against bank conflicts)
    static_assert(RB == 4 || RB == 16, "rows per workgroup");
    __shared__ uint4 stage[RB][65];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * RB;
    const int64_t tile = row0 / kTileN;
    const int rit0 = (int)(row0 % kTileN);
    if (threadIdx.x < RB && row0 + threadIdx.x < n) labels_out[row0 + threadIdx.x] = labels_in[row0 + threadIdx.x];
    uint4 *tile_base = reinterpret_cast<uint4 *>(c_bf + tile * kTileN * d_pad);
    const int64_t chunks = d_pad / 8;
    constexpr int RPW = RB / 4;   // rows per wave
    float ss[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) ss[q] = 0.f;
    for (int64_t c0 = 0; c0 < chunks; c0 += 64) {
        const int64_t j = c0 + lane;   // this lane's chunk (elements 8 j .. 8 j + 7) of each of the wave's rows
        if (j < chunks) {
            float mv[8];
            if (mu) {
                const f32x4 m0 = *reinterpret_cast<const f32x4 *>(mu + j * 8), m1 = *reinterpret_cast<const f32x4 *>(mu + j * 8 + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    mv[e] = m0[e];
                    mv[4 + e] = m1[e];
                }
            }
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int rl = w * RPW + q;
                const int64_t row = row0 + rl;
                uint16_t h[8];
                float f[8];
                if (row >= n) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        h[e] = 0;
                        f[e] = 0.f;
                    }
                } else if (j * 8 + 8 <= d) {
                    if (dtype == 0) {
                        const float *src = reinterpret_cast<const float *>(entries) + row * d + j * 8;
                        const f32x4 v0 = *reinterpret_cast<const f32x4_any *>(src), v1 = *reinterpret_cast<const f32x4_any *>(src + 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            f[e] = v0[e];
                            f[4 + e] = v1[e];
                        }
#pragma unroll
                        for (int e = 0; e < 8; ++e) h[e] = bf16_rne(f[e]);
                    } else {
                        const u32x4 wv = *reinterpret_cast<const u32x4_any *>(reinterpret_cast<const uint16_t *>(entries) + row * d + j * 8);
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            h[2 * e] = (uint16_t)(wv[e] & 0xffffu);
                            h[2 * e + 1] = (uint16_t)(wv[e] >> 16);
                        }
#pragma unroll
                        for (int e = 0; e < 8; ++e) f[e] = 0.f;   // (fp32 rows are kept only for fp32 input)
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int64_t i = j * 8 + e;
                        f[e] = 0.f;
                        h[e] = 0;
                        if (i < d) {
                            if (dtype == 0) {
                                f[e] = reinterpret_cast<const float *>(entries)[row * d + i];
                                h[e] = bf16_rne(f[e]);
                            } else {
                                h[e] = reinterpret_cast<const uint16_t *>(entries)[row * d + i];
                            }
                        }
                    }
                }
                uint4 v;   // the stored values (bf16 input) for the row-major copy
                v.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
                v.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
                v.z = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
                v.w = (uint32_t)h[6] | ((uint32_t)h[7] << 16);
                if (row < n) {
                    if (c_rows) reinterpret_cast<uint4 *>(c_rows + row * d_pad)[j] = v;
                    if (c_f32) {
                        f32x4 o0, o1;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            o0[e] = f[e];
                            o1[e] = f[4 + e];
                        }
                        *reinterpret_cast<f32x4 *>(c_f32 + row * d_pad + j * 8) = o0;
                        *reinterpret_cast<f32x4 *>(c_f32 + row * d_pad + j * 8 + 4) = o1;
                    }
                    if (mu) {
                        // the matrix cores' copy relative to mu (all zeros unless the cache is centred: then exact)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float stored = dtype == 0 ? f[e] : bf16_to_f32(h[e]);
                            h[e] = j * 8 + e < d ? bf16_rne(stored - mv[e]) : (uint16_t)0;
                        }
                        v.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
                        v.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
                        v.z = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
                        v.w = (uint32_t)h[6] | ((uint32_t)h[7] << 16);
                    }
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = bf16_to_f32(h[e]);
                    ss[q] = __builtin_fmaf(x, x, ss[q]);
                }
                stage[rl][lane] = v;
            }
        }
        __syncthreads();
        // out in tiled order: for one k-block (4 chunks) the RB rows of the block are RB * 64 bytes in a
        // row; a wave writes 64 / (4 RB) k-blocks at a time
        const int64_t kb0 = c0 / 4;
        constexpr int KPW = 64 / (4 * RB);
        for (int qb = w * KPW + lane / (4 * RB); qb < 16 && (kb0 + qb) * 4 < chunks; qb += 4 * KPW) {
            const int rl = (lane >> 2) % RB, c = lane & 3;
            tile_base[tiled_chunk_offset(rit0 + rl, (kb0 + qb) * 4 + c, kTileN)] = stage[rl][qb * 4 + c];
        }
        __syncthreads();
    }
    // |c|^2 of the bf16 row: the lanes' partial sums in a fixed order
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        float v = ss[q];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        const int64_t row = row0 + w * RPW + q;
        if (lane == 0) norm[row] = (row < n) ? v : __builtin_inff();
    }
}

hipError_t launch_cache_build(const void *entries, int dtype, int64_t n, int64_t d, int64_t n_pad, int64_t d_pad,
                              uint16_t *c_bf, float *norm, float *c_f32, uint16_t *c_rows, const int32_t *labels_in,
                              int32_t *labels_out, float *mu, double *stats, int centre_mode, hipStream_t s)
{
    hipError_t e;
    if (mu) {
        // column statistics -> mu (zeros unless the cache is to be centred)
        if ((e = launch_fill_i32(reinterpret_cast<int32_t *>(stats), 0, 4 * d_pad, s)) != hipSuccess) return e;
        const int64_t ns = n < kStatRows ? n : kStatRows;   // sampled rows
        const int64_t col_blocks = (d + 511) / 512;
        // 256 workgroups, at least 128 rows each: every workgroup ends with 1,024 fp64 atomic additions (with 512
        // workgroups of four waves 8,192 x 517 fp32 sampled took 45 us, 25 so; 8,191 and 2,047 values of bf16 99 in the mean, 62)
        int64_t row_chunks = 256 / col_blocks;
        if (row_chunks > (ns + 127) / 128) row_chunks = (ns + 127) / 128;
        if (row_chunks < 1) row_chunks = 1;
        if (row_chunks > 65535) row_chunks = 65535;
        hipLaunchKernelGGL(col_stats_kernel, dim3((unsigned)col_blocks, (unsigned)row_chunks), dim3(64 * kStatWaves), 0, s, entries,
                           dtype, n, d, d_pad, ns, stats);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(col_mean_kernel, dim3(1), dim3(1024), 0, s, stats, ns, d, d_pad, centre_mode, mu);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    static_assert(kTileN % 16 == 0, "a workgroup's rows lie in one tile");
    if (n_pad / 16 >= 512)
        hipLaunchKernelGGL(cache_build_kernel<16>, dim3((unsigned)(n_pad / 16)), dim3(256), 0, s, entries, dtype, n, d, d_pad,
                           c_bf, norm, c_f32, c_rows, mu, labels_in, labels_out);
    else
        hipLaunchKernelGGL(cache_build_kernel<4>, dim3((unsigned)(n_pad / 4)), dim3(256), 0, s, entries, dtype, n, d, d_pad,
                           c_bf, norm, c_f32, c_rows, mu, labels_in, labels_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Query preparation: bf16 copy (round to nearest even) of the live queries for the matrix
// cores in the tiled layout (tiles of bm rows), gathered through the miss list when there is
// one; rows up to the next tile boundary are zero filled.  One block per pair of rows: in the
// tiled layout the 64-byte pieces of two neighbouring rows share a 128-byte line, so eight
// consecutive threads (two rows x four 16-byte chunks of one k-block) write a whole line.
// With few rows and long activations the grid's second dimension cuts the row pair into ranges
// of chunks, so that a batch of 256 rows still fills the chip.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void query_prep_kernel(const float *queries, const int32_t *sel, const int32_t *count,
                                                         int b, int bm, int64_t d, int64_t d_pad, uint16_t *q_bf,
                                                         int32_t *flag_count, int32_t *tickets, const float *mu)
{
    const int nq = count ? *count : b;
    const int row0 = blockIdx.x * 2;   // bm is even: both rows lie in one tile
    // counters of the kernels that follow in this look-up (the list of flagged queries, the exact
    // scan's tickets) start at zero
    if (blockIdx.y == 0 && threadIdx.x < kFlagCounts) {
        if (threadIdx.x < 2 && tickets && row0 + (int)threadIdx.x < b) tickets[row0 + threadIdx.x] = 0;
        if (flag_count && blockIdx.x == 0) flag_count[threadIdx.x] = 0;
    }
    const int live_pad = ((nq + bm - 1) / bm) * bm;
    if (row0 >= live_pad) return;
    uint4 *tile_base = reinterpret_cast<uint4 *>(q_bf + (int64_t)(row0 / bm) * bm * d_pad);
    const int rsel = (threadIdx.x >> 2) & 1;
    const int row = row0 + rsel, rit = row % bm;
    const float *src = (row < nq) ? queries + (int64_t)(sel ? sel[row] : row) * d : nullptr;
    const int64_t pair_chunks = d_pad / 4;   // 16-byte chunks of the two rows together
    const int64_t per = ((pair_chunks + gridDim.y - 1) / gridDim.y + 255) / 256 * 256;   // chunks per block of the pair
    const int64_t jj_end = (blockIdx.y + 1) * per < pair_chunks ? (blockIdx.y + 1) * per : pair_chunks;
    // one 16-byte chunk of the bf16 copy from 8 fp32 values
    // (relative to the cache's mean vector when the cache is centred; mu is zero past d and all zeros
    // when it is not)
    auto convert_store = [&](int64_t j, const float (&x)[8]) {
        uint16_t h[8];
        if (mu && src) {
            const f32x4 m0 = *reinterpret_cast<const f32x4 *>(mu + j * 8);
            const f32x4 m1 = *reinterpret_cast<const f32x4 *>(mu + j * 8 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                h[e] = bf16_rne(x[e] - m0[e]);
                h[4 + e] = bf16_rne(x[4 + e] - m1[e]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) h[e] = bf16_rne(x[e]);
        }
        uint4 v;
        v.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        v.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
        v.z = (uint32_t)h[4] | ((uint32_t)h[5] << 16);
        v.w = (uint32_t)h[6] | ((uint32_t)h[7] << 16);
        tile_base[tiled_chunk_offset(rit, j, bm)] = v;
    };
    int64_t jj = blockIdx.y * per + threadIdx.x;
    // four steps' loads are issued before the first is
    // converted, so that a thread keeps 128 bytes of reads in flight
    if (src) {
        const int64_t last = d / 8 - 1;   // whole chunks
        for (; jj + 3 * 256 < jj_end && ((jj + 3 * 256) >> 3) * 4 + 3 <= last; jj += 4 * 256) {
            f32x4 v0[4], v1[4];
            int64_t jc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t ju = jj + u * 256;
                jc[u] = (ju >> 3) * 4 + (ju & 3);
                v0[u] = *reinterpret_cast<const f32x4_any *>(src + jc[u] * 8);
                v1[u] = *reinterpret_cast<const f32x4_any *>(src + jc[u] * 8 + 4);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float x[8] = {v0[u][0], v0[u][1], v0[u][2], v0[u][3], v1[u][0], v1[u][1], v1[u][2], v1[u][3]};
                convert_store(jc[u], x);
            }
        }
    }
    for (; jj < jj_end; jj += 256) {
        const int64_t j = (jj >> 3) * 4 + (jj & 3);   // chunk of 8 elements within the row
        const int64_t i0 = j * 8;
        float x[8];
        if (src && i0 + 8 <= d) {
            const f32x4 v0 = *reinterpret_cast<const f32x4_any *>(src + i0);
            const f32x4 v1 = *reinterpret_cast<const f32x4_any *>(src + i0 + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = v0[e];
                x[4 + e] = v1[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = (src && i0 + e < d) ? src[i0 + e] : 0.f;
        }
        convert_store(j, x);
    }
}

hipError_t launch_query_prep(const float *queries, const int32_t *sel, const int32_t *count, int64_t b,
                             int64_t b_pad, int bm, int64_t d, int64_t d_pad, uint16_t *q_bf, int32_t *flag_count,
                             int32_t *tickets, const float *mu, hipStream_t s)
{
    if (bm % 2 != 0 || b_pad % 2 != 0) return hipErrorInvalidValue;
    // about 2048 blocks in all, at least four rounds of 256 chunks each
    const int64_t pairs = b_pad / 2, rounds = d_pad / 4 / 256;
    int64_t ysplit = pairs > 0 ? 2048 / pairs : 1;
    if (ysplit > rounds / 4) ysplit = rounds / 4;
    if (ysplit < 1) ysplit = 1;
    hipLaunchKernelGGL(query_prep_kernel, dim3((unsigned)pairs, (unsigned)ysplit), dim3(256), 0, s, queries, sel, count,
                       (int)b, bm, d, d_pad, q_bf, flag_count, tickets, mu);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Finishing kernel, one block per live query:
//  1. gather the query's n_splits * r packed (ordered key, index) candidates and sort them
//     (bitonic, in LDS); the first r are the coarse candidates;
//  2. exact re-scoring: dist = sum_i (q_i - c_i)^2 in fp32 against the stored cache values
//     (bf16 rows widen exactly; fp32 rows when the cache was given in fp32);
//  3. rank the r candidates by (dist, index), emit the first k (Sec. 3: the k (label,
//     distance) tuples);
//  4. vote: occurrences m of each label among the k, winner = most occurrences, smaller
//     label id on equal counts; hit iff m >= vote_threshold (Sec. 2.1 / Sec. 3).
//     With the distance-weighted rule of Sec. 3 instead: C_i = (m_i / k) * sum_j 1/d_j over the
//     label's neighbours (d = square root of the reported squared distance, sums in fp64 in
//     neighbour order), winner = largest C_i, smaller label id on equality; the confidence is
//     reported in fp32 and the look-up is a hit iff it is strictly greater than the layer's
//     threshold (Pseudocode 1, FreezeInference).  A zero distance gives +inf, i.e. a hit.
// ---------------------------------------------------------------------------------------
// Exact re-scoring by one wave of `nwaves`: candidates c0 .. c0+G-1 (c0 = wave * G, stepping nwaves * G), the 64
// lanes striding over the activation 8 elements at a time; dist = sum (q_i - c_i)^2 in fp32,
// per-lane partial sums in index order, then a butterfly over the lanes (fixed order).
template <int G>
__device__ __forceinline__ void rescore_wave(const FinishArgs &a, const float *qrow, const int32_t *idx_s,
                                             float *dist_s, int r, int wave, int lane, int nwaves = 4)
{
    const bool vec = (a.d % 8) == 0;
    for (int c0 = wave * G; c0 < r; c0 += nwaves * G) {
        float acc[G];
        int64_t cand[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            acc[j] = 0.f;
            cand[j] = idx_s[(c0 + j < r) ? c0 + j : r - 1];
        }
        if (vec) {
            for (int64_t i = (int64_t)lane * 8; i < a.d; i += 64 * 8) {
                const f32x4 q0 = *reinterpret_cast<const f32x4 *>(qrow + i);
                const f32x4 q1 = *reinterpret_cast<const f32x4 *>(qrow + i + 4);
                const float qv[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
                if (a.c_f32) {
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        const float *c = a.c_f32 + cand[j] * a.d_pad + i;
                        const f32x4 c0v = *reinterpret_cast<const f32x4 *>(c);
                        const f32x4 c1v = *reinterpret_cast<const f32x4 *>(c + 4);
                        const float cv[8] = {c0v[0], c0v[1], c0v[2], c0v[3], c1v[0], c1v[1], c1v[2], c1v[3]};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float df = qv[e] - cv[e];
                            acc[j] = __builtin_fmaf(df, df, acc[j]);
                        }
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < G; ++j) {
                        const uint4 cb = *reinterpret_cast<const uint4 *>(a.c_rows + cand[j] * a.d_pad + i);
                        const uint32_t wv[4] = {cb.x, cb.y, cb.z, cb.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float c_lo = __uint_as_float(wv[e] << 16);
                            const float c_hi = __uint_as_float(wv[e] & 0xffff0000u);
                            const float d0 = qv[2 * e] - c_lo;
                            acc[j] = __builtin_fmaf(d0, d0, acc[j]);
                            const float d1 = qv[2 * e + 1] - c_hi;
                            acc[j] = __builtin_fmaf(d1, d1, acc[j]);
                        }
                    }
                }
            }
        } else {
            // Rows of another length: chain l of 64 takes elements l, l + 64, ..  fp32: a chain per lane, a few steps'
            // loads of all rows before the first is used (20,000 x 4,101, 1,100 queries: whole look-ups 694 -> 414 us).
            constexpr int U = G <= 4 ? 4 : 2;
#pragma unroll
            for (int j = 0; j < G; ++j) cand[j] = __builtin_amdgcn_readfirstlane((int32_t)cand[j]);   // (uniform: the wave's rows)
            if (a.c_f32) {   // uniform
                auto steps = [&](int64_t i, auto count) {
                    constexpr int N = decltype(count)::value;
                    float qv[N], cv[G][N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        qv[u] = qrow[i + u * 64];
#pragma unroll
                        for (int j = 0; j < G; ++j) cv[j][u] = a.c_f32[cand[j] * a.d_pad + i + u * 64];
                    }
#pragma unroll
                    for (int u = 0; u < N; ++u)
#pragma unroll
                        for (int j = 0; j < G; ++j) {
                            const float df = qv[u] - cv[j][u];
                            acc[j] = __builtin_fmaf(df, df, acc[j]);
                        }
                };
                int64_t i = lane;
                for (; i + (U - 1) * 64 < a.d; i += U * 64) steps(i, std::integral_constant<int, U>{});
                for (; i < a.d; i += 64) steps(i, std::integral_constant<int, 1>{});
            } else {
                // bf16: half a wave per row, chains 2 p and 2 p + 1 in lane p of the half, so that a lane's load is 4 bytes
                // (39 x 27,486, 11,169 queries: 5,298 us with a chain per lane and 2-byte loads).  Elements past d are zeros on
                // both sides and leave a chain as it is.
                constexpr int P = (G + 1) / 2;   // pairs of rows
                const int p = lane & 31, hf = lane >> 5;
                const uint32_t *row[P];
                float ch[P][2];
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    const int64_t lo = cand[2 * j], hi = cand[2 * j + 1 < G ? 2 * j + 1 : 2 * j];
                    row[j] = reinterpret_cast<const uint32_t *>(a.c_rows + (hf ? hi : lo) * a.d_pad) + p;
                    ch[j][0] = ch[j][1] = 0.f;
                }
                auto steps = [&](int64_t i0, auto count) {   // elements [i0, i0 + 64 N), i0 + 64 N <= d_pad
                    constexpr int N = decltype(count)::value;
                    float qv[N][2];
                    uint32_t cv[P][N];
#pragma unroll
                    for (int u = 0; u < N; ++u) {
                        const int64_t i = i0 + u * 64 + 2 * p;
#pragma unroll
                        for (int h = 0; h < 2; ++h) qv[u][h] = i + h < a.d ? qrow[i + h] : 0.f;
#pragma unroll
                        for (int j = 0; j < P; ++j) cv[j][u] = row[j][(i0 >> 1) + u * 32];
                    }
#pragma unroll
                    for (int u = 0; u < N; ++u)
#pragma unroll
                        for (int j = 0; j < P; ++j) {
                            const float d0 = qv[u][0] - __uint_as_float(cv[j][u] << 16);
                            ch[j][0] = __builtin_fmaf(d0, d0, ch[j][0]);
                            const float d1 = qv[u][1] - __uint_as_float(cv[j][u] & 0xffff0000u);
                            ch[j][1] = __builtin_fmaf(d1, d1, ch[j][1]);
                        }
                };
                int64_t i0 = 0;
                for (; i0 + U * 64 <= a.d_pad; i0 += U * 64) steps(i0, std::integral_constant<int, U>{});
                for (; i0 < a.d_pad; i0 += 64) steps(i0, std::integral_constant<int, 1>{});
                // the butterfly below, over chains 32, 16, 8, 4, 2 and 1 apart: lanes 16, 8, 4, 2 and 1 apart within the
                // half, then the lane's two chains
#pragma unroll
                for (int j = 0; j < P; ++j) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int off = 16; off >= 1; off >>= 1) ch[j][h] += __shfl_xor(ch[j][h], off, 64);
                    const int c = c0 + 2 * j + hf;
                    if (p == 0 && 2 * j + hf < G && c < r) dist_s[c] = ch[j][0] + ch[j][1];
                }
                continue;
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            float v = acc[j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == 0 && c0 + j < r) dist_s[c0 + j] = v;
        }
    }
}

// Exact re-scoring of many candidates against a short activation (d_pad <= 1024, d a multiple
// of 8) by one wave of `nwaves`: the query stays in registers (a lane owns elements 8 l .. 8 l + 7
// and 512 + 8 l .. 512 + 8 l + 7), and G candidate rows are fetched at a time, all loads issued
// before the first is used.  Same per-lane order of additions and the same butterfly as
// rescore_wave, so the same distances bit for bit.
template <int G, bool F32>
__device__ __forceinline__ void rescore_short(const FinishArgs &a, const float *qrow, const int32_t *idx_s,
                                              float *dist_s, int m, int wave, int lane, int nwaves)
{
    const int64_t i0 = (int64_t)lane * 8, i1 = i0 + 512;
    const bool h0 = i0 < a.d, h1 = i1 < a.d;
    float qv[2][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        qv[0][e] = h0 ? qrow[i0 + e] : 0.f;
        qv[1][e] = h1 ? qrow[i1 + e] : 0.f;
    }
    for (int c0 = wave * G; c0 < m; c0 += nwaves * G) {
        float acc[G];
        if constexpr (F32) {
            f32x4 cv[G][2][2];
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const float *row = a.c_f32 + (int64_t)idx_s[(c0 + j < m) ? c0 + j : m - 1] * a.d_pad;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool live = h ? h1 : h0;
                    const float *src = row + (h ? i1 : i0);
                    cv[j][h][0] = live ? *reinterpret_cast<const f32x4 *>(src) : f32x4{0.f, 0.f, 0.f, 0.f};
                    cv[j][h][1] = live ? *reinterpret_cast<const f32x4 *>(src + 4) : f32x4{0.f, 0.f, 0.f, 0.f};
                }
            }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                acc[j] = 0.f;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float df = qv[h][e] - cv[j][h][e >> 2][e & 3];
                        acc[j] = __builtin_fmaf(df, df, acc[j]);
                    }
            }
        } else {
            uint4 cb[G][2];
#pragma unroll
            for (int j = 0; j < G; ++j) {
                const uint16_t *row = a.c_rows + (int64_t)idx_s[(c0 + j < m) ? c0 + j : m - 1] * a.d_pad;
                cb[j][0] = h0 ? *reinterpret_cast<const uint4 *>(row + i0) : uint4{0, 0, 0, 0};
                cb[j][1] = h1 ? *reinterpret_cast<const uint4 *>(row + i1) : uint4{0, 0, 0, 0};
            }
#pragma unroll
            for (int j = 0; j < G; ++j) {
                acc[j] = 0.f;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t wv[4] = {cb[j][h].x, cb[j][h].y, cb[j][h].z, cb[j][h].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float c_lo = __uint_as_float(wv[e] << 16);
                        const float c_hi = __uint_as_float(wv[e] & 0xffff0000u);
                        const float d0 = qv[h][2 * e] - c_lo;
                        acc[j] = __builtin_fmaf(d0, d0, acc[j]);
                        const float d1 = qv[h][2 * e + 1] - c_hi;
                        acc[j] = __builtin_fmaf(d1, d1, acc[j]);
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < G; ++j) {
            float v = acc[j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            if (lane == 0 && c0 + j < m) dist_s[c0 + j] = v;
        }
    }
}

// Exact re-scoring by the whole block of NT threads for long activations, up to RG candidates at
// once (r <= RG, RG a multiple of 8).  The loop over the activation is the outer one: a thread
// reads its 8-element pieces of the query row once and applies each to all candidates (a 256 KB
// query row of a 64 x 32 x 32 activation does not survive in L2 between passes while the candidate
// rows stream through it: with the row re-read per eight candidates a tenth of the traffic was
// those re-reads), at the price of RG accumulators per thread.  Small batches use 1024-thread
// blocks so that a block per query still fills the memory system.  Same arithmetic as
// rescore_wave: per-thread partial sums in index order, a butterfly over the lanes, then the waves'
// sums combined in a fixed order.
// BATCHED: fp32 rows four at a time, all their loads ahead of the first use.  1,066 queries x 38,673 x 22,128, width 32: whole
// look-ups 2,227 us without, 2,087 with; width 64, i.e. two passes of 32, 3,000 x 286 x 44,976: 3,024 without, 4,294 with
// (workgroups that drift apart share less of L2).
// GS: rows whose loads are in flight at once; fewer than eight where fewer are asked for (RG = GS).
// PARTS > 1: part `part` of the order that PARTS * NT threads have, their chains part * NT .. + NT; parts are added up in turn.
template <int NT, int RG, bool BATCHED = false, int GS = 8, int PARTS = 1>
__device__ __forceinline__ void rescore_block_all(const FinishArgs &a, const float *qrow, const int32_t *idx_s,
                                                  float *dist_s, float (*red)[8], int r, int tid, int part = 0)
{
    float acc[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) acc[j] = 0.f;
    for (int64_t i = (int64_t)(PARTS > 1 ? part * NT + tid : tid) * 8; i < a.d; i += PARTS * NT * 8) {
        const f32x4 q0 = *reinterpret_cast<const f32x4 *>(qrow + i);
        const f32x4 q1 = *reinterpret_cast<const f32x4 *>(qrow + i + 4);
        const float qv[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
#pragma unroll
        for (int g = 0; g < RG; g += GS) {
            if (g < r) {   // uniform
                if (BATCHED && a.c_f32) {
#pragma unroll
                    for (int j0 = 0; j0 < 8; j0 += 4) {
                        f32x4 cv[4][2];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float *c = a.c_f32 + (int64_t)idx_s[(g + j0 + j < r) ? g + j0 + j : r - 1] * a.d_pad + i;
                            cv[j][0] = *reinterpret_cast<const f32x4 *>(c);
                            cv[j][1] = *reinterpret_cast<const f32x4 *>(c + 4);
                        }
                        __builtin_amdgcn_sched_barrier(0);   // four rows' loads leave before the first is used
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float df = qv[e] - cv[j][e >> 2][e & 3];
                                acc[g + j0 + j] = __builtin_fmaf(df, df, acc[g + j0 + j]);
                            }
                    }
                } else if (a.c_f32) {
#pragma unroll
                    for (int j = 0; j < GS; ++j) {
                        const float *c = a.c_f32 + (int64_t)idx_s[(g + j < r) ? g + j : r - 1] * a.d_pad + i;
                        const f32x4 c0v = *reinterpret_cast<const f32x4 *>(c);
                        const f32x4 c1v = *reinterpret_cast<const f32x4 *>(c + 4);
                        const float cv[8] = {c0v[0], c0v[1], c0v[2], c0v[3], c1v[0], c1v[1], c1v[2], c1v[3]};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float df = qv[e] - cv[e];
                            acc[g + j] = __builtin_fmaf(df, df, acc[g + j]);
                        }
                    }
                } else {
                    uint4 cb[GS];
#pragma unroll
                    for (int j = 0; j < GS; ++j)
                        cb[j] = *reinterpret_cast<const uint4 *>(a.c_rows + (int64_t)idx_s[(g + j < r) ? g + j : r - 1] * a.d_pad + i);
#pragma unroll
                    for (int j = 0; j < GS; ++j) {
                        const uint32_t wv[4] = {cb[j].x, cb[j].y, cb[j].z, cb[j].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float c_lo = __uint_as_float(wv[e] << 16);
                            const float c_hi = __uint_as_float(wv[e] & 0xffff0000u);
                            const float d0 = qv[2 * e] - c_lo;
                            acc[g + j] = __builtin_fmaf(d0, d0, acc[g + j]);
                            const float d1 = qv[2 * e + 1] - c_hi;
                            acc[g + j] = __builtin_fmaf(d1, d1, acc[g + j]);
                        }
                    }
                }
            }
        }
    }
#pragma unroll
    for (int g = 0; g < RG; g += GS) {
        if (g < r) {   // uniform
#pragma unroll
            for (int j = 0; j < GS; ++j) {
                float v = acc[g + j];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
                if ((tid & 63) == 0) red[tid >> 6][j] = v;
            }
            __syncthreads();
            if (tid < GS && g + tid < r) {
                float t = PARTS > 1 && part > 0 ? dist_s[g + tid] : 0.f;
#pragma unroll
                for (int wv = 0; wv < NT / 64; wv += 4)   // fixed order: groups of four waves
                    t += (red[wv][tid] + red[wv + 1][tid]) + (red[wv + 2][tid] + red[wv + 3][tid]);
                dist_s[g + tid] = t;
            }
            __syncthreads();
        }
    }
}

// The same by 256 threads in the order that the batch's finishing kernel has (wide_order): a distance does not depend on
// whether the first candidates confirmed the query.
template <int RG>
__device__ __forceinline__ void rescore_block_any(const FinishArgs &a, const float *qrow, const int32_t *idx_s, float *dist_s, float (*red)[8],
                                                  int r, int tid)
{
    if (wide_order(a.b, a.d)) {   // uniform
        for (int part = 0; part < 4; ++part) rescore_block_all<256, RG, false, 8, 4>(a, qrow, idx_s, dist_s, red, r, tid, part);
    } else {
        rescore_block_all<256, RG>(a, qrow, idx_s, dist_s, red, r, tid);
    }
}

// Label and hit decision from the k nearest neighbours (labels lab_s[k], squared distances
// dsel_s[k], nearest first), by the first k threads of the block; cnt_s / conf_s are scratch.
// Plurality rule: occurrences m of each label, winner = most occurrences, smaller label id on
// equal counts, hit iff m >= vote_threshold.  Distance-weighted rule of Sec. 3: C_i = (m_i / k) *
// sum_j 1 / d_j in fp64 in neighbour order, winner = largest C_i (smaller id on equality), the
// confidence rounded once to fp32, hit iff confidence > threshold (Pseudocode 1).
// k-means cache (Sec. 4; k = 1): the label is the nearest centre's majority label and the
// confidence its majority share over the distance (zero distance: +inf, or 0 for an empty cluster).
__device__ __forceinline__ void decide_and_write(const FinishArgs &a, int q, int tid, const int32_t *lab_s,
                                                 const float *dsel_s, int32_t *cnt_s, double *conf_s, int32_t nearest)
{
    if (a.weighted == 2) {
        if (tid == 0) {
            const double fr = (double)a.fraction[nearest], dd = (double)dsel_s[0];
            const float conf = dd > 0.0 ? (float)(fr / __builtin_sqrt(dd)) : (fr > 0.0 ? __builtin_inff() : 0.f);
            a.out_labels[q] = lab_s[0];
            a.out_votes[q] = 1;
            a.out_conf[q] = conf;
            a.out_hit[q] = (uint8_t)(conf > a.conf_threshold);
        }
        return;
    }
    if (tid < a.k) {
        const int32_t lm = lab_s[tid];
        int c = 0;
        for (int j = 0; j < a.k; ++j) c += (lab_s[j] == lm);
        cnt_s[tid] = c;
        if (a.weighted == 1) {
            double inv = 0.0;
            for (int j = 0; j < a.k; ++j)
                if (lab_s[j] == lm) inv += 1.0 / __builtin_sqrt((double)dsel_s[j]);
            conf_s[tid] = ((double)c / (double)a.k) * inv;
        }
    }
    __syncthreads();
    if (tid == 0 && a.weighted == 1) {
        double best_conf = -1.0;
        int best_c = 0;
        int32_t best_l = 0;
        for (int j = 0; j < a.k; ++j) {
            const double cf = conf_s[j];
            const int32_t l = lab_s[j];
            if (cf > best_conf || (cf == best_conf && l < best_l)) {
                best_conf = cf;
                best_l = l;
                best_c = cnt_s[j];
            }
        }
        const float conf = (float)best_conf;
        a.out_labels[q] = best_l;
        a.out_votes[q] = best_c;
        a.out_conf[q] = conf;
        a.out_hit[q] = (uint8_t)(conf > a.conf_threshold);
    } else if (tid == 0) {
        int best_c = 0;
        int32_t best_l = 0;
        for (int j = 0; j < a.k; ++j) {
            const int c = cnt_s[j];
            const int32_t l = lab_s[j];
            if (c > best_c || (c == best_c && l < best_l)) {
                best_c = c;
                best_l = l;
            }
        }
        a.out_labels[q] = best_l;
        a.out_votes[q] = best_c;
        a.out_hit[q] = (uint8_t)(best_c >= a.vote_threshold);
    }
}

// Rank of each of the m re-scored candidates under (distance, index); the first k go to the
// outputs and to lab_s / dsel_s.  Also counts the candidates that are not preceded by one at the
// same distance (*distinct_s, zero on entry): how many different samples the certificate has.
__device__ __forceinline__ void rank_and_emit(const FinishArgs &a, int q, int m, int tid, int nthreads, const float *dist_s,
                                              const int32_t *idx_s, int32_t *lab_s, float *dsel_s, int32_t *nearest_s,
                                              int *distinct_s)
{
    for (int c = tid; c < m; c += nthreads) {
        const float dm = dist_s[c];
        const int32_t im = idx_s[c];
        int rank = 0, twin = 0;
        for (int j = 0; j < m; ++j) {
            const float dj = dist_s[j];
            const int32_t ij = idx_s[j];
            rank += (dj < dm) || (dj == dm && ij < im);
            twin |= (dj == dm && ij < im);
        }
        if (!twin) atomicAdd(distinct_s, 1);
        if (rank < a.k) {
            a.out_nbr_idx[(int64_t)q * a.k + rank] = im;
            a.out_nbr_dist[(int64_t)q * a.k + rank] = dm;
            lab_s[rank] = a.labels[im];
            dsel_s[rank] = dm;
            if (rank == 0) *nearest_s = im;
        }
    }
}

// The gathered candidates of query q in ent (marker-padded to a power of two); returns how many slots
// they take.  *real_s = real cache entries among them; *excl_s = a lower bound (ordered bits) of the keys of
// all entries that were not gathered (valid when the candidates are per-split lists; else the marker).
__device__ __forceinline__ int gather_entries(const FinishArgs &a, int q, int nq, uint64_t *ent, int *real_s, uint32_t *excl_s,
                                              int tid, int nthreads)
{
    const int r = a.r;
    int n_splits = a.n_splits;
    if (a.count && !a.part_count)   // cascade: the distance pass derived its splits from the live count
        n_splits = splits_for((nq + a.bm - 1) / a.bm, a.n_tiles, a.num_cus, a.max_splits);
    int total = n_splits * r, stride = a.alloc_splits * r;
    if (a.part_count) {
        stride = a.part_stride;
        total = a.part_count[q] < stride ? a.part_count[q] : stride;
    }
    int sort_n = 2;
    while (sort_n < total) sort_n <<= 1;
    const uint64_t *src = a.part + (size_t)q * stride;
    if (tid == 0) {
        *real_s = 0;
        *excl_s = 0xffffffffu;
    }
    __syncthreads();
    int mine = 0;
    for (int i = tid; i < sort_n; i += nthreads) {
        const uint64_t x = (i < total) ? src[i] : kSentinel;
        ent[i] = x;
        mine += (uint32_t)x < (uint32_t)a.n;   // a real cache entry (the "no entry" marker carries index 2^32 - 1)
    }
    if (mine) atomicAdd(real_s, mine);
    __syncthreads();
    if (!a.part_count && *real_s < a.n) {   // uniform (else nothing is left out)
        // Per-split lists: a split that filled its list kept its r smallest keys, so every entry
        // of its range that it dropped has a key >= the list's largest.  The smallest of these
        // bounds every entry outside the gathered lists.  (Slots rotate with the thread
        // number so that neighbouring threads read different LDS banks.)
        for (int sp = tid; sp < n_splits; sp += nthreads) {
            uint32_t mx = 0;
            int jj = sp % r;
            for (int j = 0; j < r; ++j) {
                const uint32_t kb = (uint32_t)(ent[sp * r + jj] >> 32);
                mx = kb > mx ? kb : mx;
                jj = jj + 1 == r ? 0 : jj + 1;
            }
            atomicMin(excl_s, mx);   // a list with an empty slot dropped nothing: its largest is the marker
        }
        __syncthreads();
    }
    return total;
}

struct FinishKernelArgs {
    FinishArgs a;
    int sort_cap;   // power of two >= the largest number of entries gathered per query (LDS allocation)
    int m_first;    // candidates re-scored at first (first_width)
};

// Exactness certificate of the bf16 pre-filter, by the first wave of the block (every thread
// calls; the verdict is valid in every thread after the call).
//
// The m candidates ent[0 .. m) (coarse key kappa_j in the upper half) were re-scored exactly
// (dist_s[j]); dk is the k-th smallest of those exact distances.  Every entry that was NOT
// re-scored has a coarse key >= the float behind excl_bits (+inf or the "no entry" marker: there is
// no such entry).
// The coarse key is the exact distance minus |q|^2 plus an error (bf16 rounding of the query, and of
// the entries when the cache is stored in fp32; fp32 accumulation), so e_j = kappa_j - dist_j
// samples (error - |q|^2) on entries as near to the query as any that could have been missed.  With
// mean and standard deviation sd of the e_j, an excluded entry has, under that error distribution,
//     distance >= kappa_excl - mean - z (1 + 4/m) sd sqrt(1 + 1/m),
// and when this exceeds dk no excluded entry can be among the k nearest: the result is the exact
// one.  z = kCertZ; the estimate needs kCertMinSamples samples from as many distinct distances
// (duplicated rows repeat one sample).  Otherwise the verdict is "unconfirmed" and the caller
// widens the candidate set or hands the query to the exact scan.  Two calls with the same verdict_s want a
// barrier between them.
// floor_ulps: the margin is at least this many fp32 ulps of the quantities involved (ties; rounding that the
// samples do not show).
__device__ __forceinline__ bool certificate(const uint64_t *ent, const float *dist_s, int m, float dk, uint32_t excl_bits,
                                            int distinct, int tid, int *verdict_s, double floor_ulps = 4.0)
{
    if (tid < 64) {
        const double e0 = (double)from_ordered_bits((uint32_t)(ent[0] >> 32)) - (double)dist_s[0];
        double s1 = 0.0, s2 = 0.0;
        for (int j = tid; j < m; j += 64) {
            const double e = ((double)from_ordered_bits((uint32_t)(ent[j] >> 32)) - (double)dist_s[j]) - e0;
            s1 += e;
            s2 += e * e;
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            s1 += __shfl_xor(s1, off, 64);
            s2 += __shfl_xor(s2, off, 64);
        }
        if (tid == 0) {
            int ok;
            if (excl_bits >= 0xff800000u) {
                ok = 1;   // nothing was left out (marker), or only padding rows (their keys are +inf)
            } else if (m < kCertMinSamples || distinct < kCertMinSamples) {
                ok = 0;
            } else {
                const double mean_rel = s1 / m;
                double var = (s2 - m * mean_rel * mean_rel) / (m - 1);
                var = var > 0.0 ? var : 0.0;
                const double mean = e0 + mean_rel;
                const double kex = (double)from_ordered_bits(excl_bits);
                // z standard deviations of (an excluded entry's error minus the sample mean), widened by
                // 1 + 4/m for the uncertainty of a standard deviation estimated from m samples
                double margin = kCertZ * (1.0 + 4.0 / m) * __builtin_sqrt(var * (1.0 + 1.0 / m));
                const double floor_ = floor_ulps * 5.9604644775390625e-8 * (__builtin_fabs(kex) + __builtin_fabs(mean) + (double)dk);
                margin = margin > floor_ ? margin : floor_;
                ok = (kex - mean - margin > (double)dk) ? 1 : 0;   // false for NaN
            }
            *verdict_s = ok;
        }
    }
    __syncthreads();
    return *verdict_s != 0;
}

// Candidates re-scored in a first step; the others of the r only for the queries that these do not confirm.  Long
// rows only: they are what the finishing kernels wait for.
//   - three quarters of a width that leaves room (16 with k <= 10, 32 with k <= 20, 64 with k <= 40): 92 % of the queries of
//     10,000 x 50,000 x 8,192, k = 10, are spared the last four rows (0.42 -> 0.36 ms for the batch).  `quarter` false: not
//     this one (few queries: fetching the last quarter at once costs less than a second round of latency);
//   - of a wider width than k has by default the default: 256 queries x 50,000 x 65,536, k = 10, width 64, 1,830 -> 1,621 us the
//     whole look-up.
__host__ __device__ inline int first_width(const FinishArgs &a, bool quarter)
{
    if (a.d < 4096 || a.d % 8 != 0) return a.r;
    const int own = a.k <= 10 ? 16 : (a.k <= 24 ? 32 : 64);
    if (a.r > own) return own;
    return quarter && a.r == own && a.k <= own / 2 + own / 8 ? own - own / 4 : a.r;
}

// 256-thread blocks are held to four waves per SIMD, i.e. at most 128 registers: the compiler
// would take 169 and leave two blocks per CU, too few to cover one block's merge and final
// phases with the other blocks' re-scoring loads (0.55 -> 0.45 ms on 10,000 queries x 8,192).
//
// One block per live query; a query the certificate does not confirm goes on list 0, the wider
// re-scoring's (or straight on list 1, the exact scan's, when no further entries were gathered for it).
template <int NT>
__global__ __launch_bounds__(NT, NT == 256 ? 4 : 1) void finish_kernel(FinishKernelArgs fa)
{
    const FinishArgs &a = fa.a;
    extern __shared__ uint64_t ent[];   // sort_cap entries (dynamic: small merges keep occupancy high)
    __shared__ float red[NT / 64][8];
    __shared__ float dist_s[kMaxRescore];
    __shared__ int32_t idx_s[kMaxRescore];
    __shared__ int32_t lab_s[kMaxK];
    __shared__ int32_t cnt_s[kMaxK];
    __shared__ float dsel_s[kMaxK];
    __shared__ double conf_s[kMaxK];
    __shared__ int32_t nearest_s;
    __shared__ int real_s, distinct_s, verdict_s;
    __shared__ uint32_t excl_s;

    const int nq = a.count ? *a.count : a.b;
    const int tid = threadIdx.x;
    if ((int)blockIdx.x >= nq) return;   // uniform
    int q = blockIdx.x;
    if (a.order) {
        // neighbours of the order on one XCD (block id modulo 8)
        const int x8 = q & 7, a8 = nq >> 3, rem8 = nq & 7;
        q = a.order[x8 * a8 + (x8 < rem8 ? x8 : rem8) + (q >> 3)];
    }
    const int r = a.r;

    // 1. merge the per-split lists
    const int total = gather_entries(a, q, nq, ent, &real_s, &excl_s, tid, NT);
    int sort_n = 2;
    while (sort_n < total) sort_n <<= 1;   // <= fa.sort_cap, the LDS allocation
    if (tid == 0) distinct_s = 0;
    bitonic_sort_lds(ent, sort_n, tid, NT);
    const float *qrow = a.queries + (int64_t)(a.sel ? a.sel[q] : q) * a.d;
    // the others are re-scored only when the certificate over the first ones, which then counts them among the
    // excluded entries, does not confirm the result (first_width)
    const int m_first = fa.m_first;

    for (int c = tid; c < r; c += NT) {
        // With finite inputs every one of the first r entries is a real cache row.  Non-finite
        // inputs (outside the contract) can leave "no entry" markers here: map them to row 0 so
        // that nothing is read out of bounds.
        const uint32_t ci = (uint32_t)(ent[c] & 0xffffffffu);
        idx_s[c] = ci < (uint32_t)a.n ? (int32_t)ci : 0;
    }
    __syncthreads();

    // 2. exact fp32 re-scoring: each wave takes a group of candidates and needs no block barrier
    if (a.d >= 4096 && a.d % 8 == 0) {
        // long activations: the whole block per candidate, the query row read once
        if (r <= 16) {
            rescore_block_all<NT, 16, true>(a, qrow, idx_s, dist_s, red, m_first, tid);
        } else if (r <= 32) {
            rescore_block_all<NT, 32, true>(a, qrow, idx_s, dist_s, red, m_first, tid);
        } else {
            // (two passes of 32: 64 accumulators per thread spill, and the pass is 8 % slower for it)
            for (int c0 = 0; c0 < m_first; c0 += 32)
                rescore_block_all<NT, 32>(a, qrow, idx_s + c0, dist_s + c0, red, m_first - c0 < 32 ? m_first - c0 : 32, tid);
        }
    } else if (tid < 256) {   // short activations: four waves, one group of candidates each
        if (r <= 16)
            rescore_wave<4>(a, qrow, idx_s, dist_s, r, tid >> 6, tid & 63);
        else if (r <= 32)
            rescore_wave<8>(a, qrow, idx_s, dist_s, r, tid >> 6, tid & 63);
        else
            rescore_wave<16>(a, qrow, idx_s, dist_s, r, tid >> 6, tid & 63);
    }
    __syncthreads();

    // 3. final order (dist, index) and the first k
    const int real = real_s;   // real entries gathered
    const int wider = real < kTier1 ? real : kTier1;
    // the certificate: is any entry that was not re-scored possibly nearer than the k-th?
    bool ok = false;
    if (m_first < r) {
        rank_and_emit(a, q, m_first, tid, NT, dist_s, idx_s, lab_s, dsel_s, &nearest_s, &distinct_s);
        __syncthreads();
        const uint32_t nxt = (uint32_t)(ent[m_first] >> 32);   // (real >= r > m_first with finite inputs; else the marker)
        ok = certificate(ent, dist_s, m_first, dsel_s[a.k - 1], nxt < excl_s ? nxt : excl_s, distinct_s, tid, &verdict_s);
        if (!ok) {   // uniform
            rescore_block_all<NT, 16, true>(a, qrow, idx_s + m_first, dist_s + m_first, red, r - m_first, tid);
            if (tid == 0) distinct_s = 0;
            __syncthreads();
        }
    }
    if (!ok) {
        rank_and_emit(a, q, r, tid, NT, dist_s, idx_s, lab_s, dsel_s, &nearest_s, &distinct_s);
        __syncthreads();
        uint32_t excl = excl_s;
        if (real > r) {
            const uint32_t nxt = (uint32_t)(ent[r] >> 32);
            excl = nxt < excl ? nxt : excl;
        }
        ok = certificate(ent, dist_s, r, dsel_s[a.k - 1], excl, distinct_s, tid, &verdict_s);
    }
    if (tid == 0) {
        // unconfirmed: the wider round, or the exact scan, redoes this query (the outputs written
        // here stand until then)
        const int next = wider <= r ? 1 : 0;
        if (!ok) {
            const int pos = atomicAdd(a.flag_count + next, 1);
            (next ? a.flag_list2 : a.flag_list)[pos] = q;
        }
        if (a.stats && (ok || next == 1)) atomicAdd(a.stats + (ok ? 0 : 2), 1ull);
    }

    // 4. vote and hit decision
    decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
}

// ---------------------------------------------------------------------------------------
// Finishing kernel of the small-batch path (short activations, at most 16 queries), from the
// block minima alone.  One launch, grid (pairs of blocks, queries), 1024 threads:
//  1. selection (every workgroup of a query repeats it: a few thousand L2-resident reads): T =
//     the R-th smallest block minimum; the R blocks whose minimum is <= T hold every entry that is
//     <= T, hence the R best by the coarse key.  It starts from the per-workgroup minima of the
//     streaming kernel, so only the block minima of the R groups that can matter are read.  The
//     selected blocks are put in ascending order of their minima, the same in every workgroup.
//  2. workgroup x re-scores blocks 2 x and 2 x + 1 of that order exactly in fp32 (64 entries, the
//     same arithmetic as above), sorts them in one wave and leaves the `keep` nearest, and for
//     each block the (coarse key, exact distance) of its minimum entry: samples of the coarse
//     key's error for the certificate.
//  3. the last workgroup of a query to arrive (a ticket per query) takes the k nearest by
//     (distance, index) of what was left, decides label and hit, and checks the certificate:
//     every entry outside the selected blocks has a coarse key >= T.  Unconfirmed queries go on
//     the list of the exact scan.
// ---------------------------------------------------------------------------------------
struct SkinnyTailArgs {
    FinishArgs a;            // queries, cache rows, n, d, d_pad, outputs, flag list (a.r = blocks to take)
    const uint64_t *bmin;    // [b, nb] smallest (ordered key, index) of every block of 32 entries
    const uint64_t *wgmin;   // [b, n_groups] smallest value of each group of blocks
    int64_t nb;
    int n_groups, n_tiles;   // group j = the blocks of cache tiles [j n_tiles / n_groups, (j+1) n_tiles / n_groups)
    uint64_t *cand;          // [b, pairs * keep] packed (ordered distance, index), marker-padded
    uint64_t *samp;          // [b, 2 pairs] (coarse key bits << 32 | distance bits) of each block's minimum entry
    int32_t *tickets;        // [b], zero on entry (the streaming kernel clears them); left zero
    int keep;                // entries each workgroup passes on (<= 64)
    int pairs;               // workgroups per query
};

// The R-th smallest of list[0..cnt) (distinct values), cnt <= kThrList, by the whole workgroup.
__device__ inline uint64_t rth_of_list(uint64_t *list, int cnt, int r_sel, uint64_t *sel_s, int tid)
{
    if (cnt <= kThrThreads) {
        select_by_rank_counting(list, cnt, r_sel - 1, tid, sel_s);
        __syncthreads();
        return *sel_s;
    }
    int n2 = 2;
    while (n2 < cnt) n2 <<= 1;
    for (int i = cnt + tid; i < n2; i += kThrThreads) list[i] = kSentinel;
    __syncthreads();
    bitonic_sort_lds(list, n2, tid, kThrThreads);
    return list[r_sel - 1];
}

__global__ __launch_bounds__(kThrThreads) void skinny_tail_kernel(SkinnyTailArgs sa)
{
    const FinishArgs &a = sa.a;
    __shared__ uint64_t list[kThrList];
    __shared__ uint64_t gm_s[kThrThreads];
    __shared__ uint64_t pick_s[kMaxRescore];   // minima (pairs) of the selected blocks, ascending
    __shared__ uint64_t sel_s;
    __shared__ int list_n, blk_n, grp_n, last_s, distinct_s, verdict_s;
    __shared__ int32_t grp_s[kMaxRescore];
    __shared__ int32_t idx_s[64], row_s[64];
    __shared__ float dist_s[64];
    __shared__ int32_t lab_s[kMaxK], cnt_s[kMaxK];
    __shared__ float dsel_s[kMaxK];
    __shared__ double conf_s[kMaxK];
    __shared__ int32_t nearest_s;
    const int q = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    const int64_t nb = sa.nb;
    const int r = a.r;

    // ---- 1. selection ----
    int nblk;
    if (r >= nb) {   // fewer blocks than wanted: take them all, in index order
        if (tid < (int)nb) pick_s[tid] = sa.bmin[(size_t)q * nb + tid];
        nblk = (int)nb;
        __syncthreads();
    } else {
        // 1a. the groups that can hold one of the r smallest block minima: those whose own minimum
        //     is among the r smallest group minima (T1 = the r-th of them bounds the answer above)
        const int ng = sa.n_groups;
        if (tid == 0) {
            list_n = 0;
            blk_n = 0;
            grp_n = 0;
        }
        const uint64_t my_gm = tid < ng ? sa.wgmin[(size_t)q * ng + tid] : kSentinel;
        gm_s[tid] = my_gm;
        __syncthreads();
        uint64_t t1 = kSentinel;
        if (r < ng) {
            if (r <= 32) {
                t1 = smallest_sorted(gm_s, list, ng, r, tid, kThrThreads)[r - 1];
            } else {
                select_by_rank_counting(gm_s, ng, r - 1, tid, &sel_s);
                __syncthreads();
                t1 = sel_s;
            }
            __syncthreads();
        }
        if (tid < ng && my_gm <= t1) {
            const int pos = atomicAdd(&grp_n, 1);
            if (pos < kMaxRescore) grp_s[pos] = tid;
        }
        __syncthreads();
        const int ngrp = grp_n < kMaxRescore ? grp_n : kMaxRescore;   // min(r, ng) groups
        // 1b. gather their block minima <= T1: at least r, at most r * (blocks per group)
        const int bpg = ((sa.n_tiles + ng - 1) / ng) * (kTileN / 32);
        const uint64_t *src = sa.bmin + (size_t)q * nb;
        for (int c = tid; c < ngrp * bpg; c += kThrThreads) {
            const int gidx = grp_s[c / bpg];
            const int64_t b0 = ((int64_t)gidx * sa.n_tiles / ng) * (kTileN / 32);
            const int64_t b1 = ((int64_t)(gidx + 1) * sa.n_tiles / ng) * (kTileN / 32);
            const int64_t bi = b0 + c % bpg;
            if (bi < b1) {
                const uint64_t x = src[bi];
                if (x <= t1) {
                    const int pos = atomicAdd(&list_n, 1);
                    if (pos < kThrList) list[pos] = x;
                }
            }
        }
        __syncthreads();
        const int cnt = list_n < kThrList ? list_n : kThrList;
        // 1c. the r smallest of them, ascending, are the minima of the blocks to take (distinct values)
        if (r <= 32 && cnt <= kThrList / 2) {
            const uint64_t *res = smallest_sorted(list, list + kThrList / 2, cnt, r, tid, kThrThreads);
            if (tid < r) pick_s[tid] = res[tid];
        } else {
            const uint64_t t = rth_of_list(list, cnt, r, &sel_s, tid);
            __syncthreads();
            for (int i = tid; i < cnt; i += kThrThreads) {
                const uint64_t x = list[i];
                if (x <= t) {
                    const int pos = atomicAdd(&blk_n, 1);
                    if (pos < kMaxRescore) pick_s[pos] = x;
                }
            }
            __syncthreads();
            if (tid < 64) {   // exactly r <= 64 values: one wave puts them in order
                const uint64_t v = wave_sort64(lane < r ? pick_s[lane] : kSentinel, lane);
                if (lane < r) pick_s[lane] = v;
            }
        }
        nblk = r;
        __syncthreads();
    }

    // ---- 2. exact re-scoring of this workgroup's two blocks ----
    uint64_t *out = sa.cand + ((size_t)q * sa.pairs + blockIdx.x) * sa.keep;
    uint64_t *samp = sa.samp + (size_t)q * 2 * sa.pairs + 2 * blockIdx.x;
    const int first = blockIdx.x * 2;
    const int here = nblk - first < 2 ? nblk - first : 2;   // blocks of this workgroup
    if (here <= 0) {
        if (tid < sa.keep) out[tid] = kSentinel;
        if (tid < 2) samp[tid] = kSentinel;
    } else {
        const int m = here * 32;
        // entries past the cache (padding rows of the last tile) are re-scored as row 0 and dropped below
        if (tid < m) {
            const int e = (int)((uint32_t)pick_s[first + (tid >> 5)] >> 5) * 32 + (tid & 31);
            idx_s[tid] = e < a.n ? e : -1 - e;
            row_s[tid] = e < a.n ? e : 0;
        }
        __syncthreads();
        const float *qrow = a.queries + (int64_t)q * a.d;
        if (a.d % 8 != 0)
            rescore_wave<4>(a, qrow, row_s, dist_s, m, tid >> 6, lane, kThrThreads / 64);
        else if (a.c_f32)
            rescore_short<4, true>(a, qrow, row_s, dist_s, m, tid >> 6, lane, kThrThreads / 64);
        else
            rescore_short<4, false>(a, qrow, row_s, dist_s, m, tid >> 6, lane, kThrThreads / 64);
        __syncthreads();
        if (tid < 64) {
            uint64_t x = kSentinel;
            if (tid < m && idx_s[tid] >= 0) x = ((uint64_t)ordered_bits(dist_s[tid]) << 32) | (uint32_t)idx_s[tid];
            x = wave_sort64(x, lane);
            if (lane < sa.keep) out[lane] = x;
        } else if (tid < 66) {
            const int hb = tid - 64;
            uint64_t sv = kSentinel;
            if (hb < here) {
                const uint64_t pr = pick_s[first + hb];   // (coarse key, index) of the block's minimum entry
                sv = (pr & 0xffffffff00000000ull) | __float_as_uint(dist_s[hb * 32 + ((uint32_t)pr & 31u)]);
            }
            samp[hb] = sv;
        }
    }

    // ---- 3. the last workgroup of the query finishes it ----
    // (the barrier orders every thread's stores before thread 0's fence, which publishes them to the
    // device before the ticket is taken; the last workgroup reads them with device-coherent loads)
    __syncthreads();
    if (tid == 0) {
        __threadfence();
        last_s = (atomicAdd(&sa.tickets[q], 1) == sa.pairs - 1);
        __threadfence();
    }
    __syncthreads();
    if (!last_s) return;   // uniform
    const int mcand = sa.pairs * sa.keep;   // <= kThrList / 2
    for (int c = tid; c < mcand; c += kThrThreads)
        list[c] = __hip_atomic_load(sa.cand + (size_t)q * mcand + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) {
        sa.tickets[q] = 0;
        distinct_s = 0;
    }
    __syncthreads();
    const uint64_t *res;
    if (a.k <= 32) {
        res = smallest_sorted(list, list + kThrList / 2, mcand, a.k, tid, kThrThreads);
    } else {
        int n2 = 2;
        while (n2 < mcand) n2 <<= 1;
        for (int c = mcand + tid; c < n2; c += kThrThreads) list[c] = kSentinel;
        __syncthreads();
        bitonic_sort_lds(list, n2, tid, kThrThreads);
        res = list;
    }
    if (tid < a.k) {
        const uint64_t x = res[tid];
        // with finite inputs the first k are real entries; a "no entry" marker maps to row 0
        const int32_t im = x == kSentinel ? 0 : (int32_t)(uint32_t)x;
        const float dm = from_ordered_bits((uint32_t)(x >> 32));
        a.out_nbr_idx[(int64_t)q * a.k + tid] = im;
        a.out_nbr_dist[(int64_t)q * a.k + tid] = dm;
        lab_s[tid] = a.labels[im];
        dsel_s[tid] = dm;
        if (tid == 0) nearest_s = im;
    }
    __syncthreads();
    // certificate from the block minima: gm_s = the samples' coarse keys (upper halves), dist_s = their distances
    if (tid < nblk) {
        const uint64_t sv = __hip_atomic_load(sa.samp + (size_t)q * 2 * sa.pairs + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        gm_s[tid] = sv & 0xffffffff00000000ull;
        dist_s[tid] = __uint_as_float((uint32_t)sv);
    }
    __syncthreads();
    if (tid < nblk) {
        int twin = 0;
        for (int j = 0; j < tid; ++j) twin |= (dist_s[j] == dist_s[tid]);
        if (!twin) atomicAdd(&distinct_s, 1);
    }
    __syncthreads();
    const uint32_t excl = r >= nb ? 0xffffffffu : (uint32_t)(pick_s[nblk - 1] >> 32);
    const bool ok = certificate(gm_s, dist_s, nblk, dsel_s[a.k - 1], excl, distinct_s, tid, &verdict_s);
    if (tid == 0) {
        if (!ok) {
            const int pos = atomicAdd(a.flag_count + 1, 1);
            a.flag_list2[pos] = q;
        }
        if (a.stats) atomicAdd(a.stats + (ok ? 0 : 2), 1ull);
    }
    decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
}

size_t skinny_finish_workspace_bytes(int r, size_t align)
{
    auto up = [&](size_t x) { return (x + align - 1) / align * align; };
    const size_t pairs = (size_t)(r + 1) / 2;
    return up((size_t)kSkinnyRows * pairs * 64 * 8) + up((size_t)kSkinnyRows * pairs * 2 * 8);
}

hipError_t launch_skinny_finish(const FinishArgs &a, const uint64_t *bmin, const uint64_t *wgmin, int64_t nb,
                                int n_groups, int n_tiles, uint64_t *cand, uint64_t *samp, int32_t *tickets, hipStream_t s)
{
    if (a.r < 1 || a.r > kMaxRescore || a.k > kMaxK || a.k > a.r || a.b < 1 || a.b > kSkinnyRows || a.sel || a.count)
        return hipErrorInvalidValue;
    if (n_groups < 1 || n_groups > kThrThreads || n_groups > n_tiles) return hipErrorInvalidValue;
    if (!a.flag_count || !a.flag_list2 || !tickets) return hipErrorInvalidValue;
    const int64_t bpg = ((int64_t)(n_tiles + n_groups - 1) / n_groups) * (kTileN / 32);
    if (a.r < nb && bpg * a.r > kThrList) return hipErrorInvalidValue;
    const int pairs = (a.r + 1) / 2;   // a.r >= the number of blocks selected
    const int keep = a.k <= 32 ? a.k : 64;
    SkinnyTailArgs ta{a, bmin, wgmin, nb, n_groups, n_tiles, cand, samp, tickets, keep, pairs};
    hipLaunchKernelGGL(skinny_tail_kernel, dim3((unsigned)pairs, (unsigned)a.b), dim3(kThrThreads), 0, s, ta);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Finishing kernel of the keys-out routes (at most 1,024 queries): selection, exact re-scoring,
// final top-k, certificate and vote in one launch, one workgroup of 1,024 threads per query.
//  1. Selection.  The block minima are dealt into 256 groups (value j belongs to group j mod 256);
//     T = the r_sel-th smallest group minimum.  At least r_sel blocks have a minimum <= T, so at
//     least r_sel entries are <= T, and every entry <= T lies in one of those blocks: their keys
//     (128 bytes a block) give the candidates.  r_sel is twice the re-scoring width, so that a query
//     the certificate does not confirm has candidates left for the wider re-scoring.  Usually T leaves
//     few more than r_sel blocks; with more than 64, T falls to the r_sel-th smallest minimum itself.
//  2. The candidates (usually up to 64: one wave sorts them in registers) in order of their keys; the
//     first r are re-scored by all sixteen waves: rows of 16,384 values and more by the whole block,
//     from 4,096 on a quarter of the candidates by each group of four waves, shorter ones a candidate
//     per wave.  Same order of additions as in finish_kernel.
//  3. As in finish_kernel.
// A dependent launch costs about 6 us here and the serial chain of small steps is what bounds the rest.
// A 1,024-thread kernel for the selection and finish_kernel after it took 11 + 28 us on 32 queries x
// 50,000 x 8,192 and 11 + 10 us on 256 x 2,000 x 512 (whole look-ups 203 and 35.9 us); this kernel takes 19
// and 11 us (185 and 26.0 us).
// ---------------------------------------------------------------------------------------
struct KeysFinishArgs {
    FinishArgs a;
    const uint64_t *bmin;   // [b, nb] smallest (ordered key, index) of every block of 32 entries
    const float *keys;      // [b, n_pad]
    int64_t nb, n_pad;
    int r_sel;              // blocks the threshold lets in at least (<= kMaxRescore)
    uint64_t *cand;         // [b, a.part_stride] candidates left for the wider re-scoring of an unconfirmed query
    int32_t *cand_count;    // [b]
    int m_first;            // candidates re-scored at first (first_width)
    int parts;              // workgroups that share a query's first re-scoring
    float *meet;            // [b, kMaxRescore] (parts > 1) their distances
    int32_t *tickets;       // [b] (parts > 1) zero on entry; left zero
};

// dist_s[0 .. m) for rows of d values (a multiple of 8), 1,024 threads: group g of four waves takes
// candidates g * per .. (RG of them at most); per-thread sums, butterfly and the sum over the four waves as in
// rescore_block_all<256, .>.
template <int RG>
__device__ __forceinline__ void rescore_groups(const FinishArgs &a, const float *qrow, const int32_t *idx_s, float *dist_s,
                                               float (*red)[RG], int m, int tid)
{
    const int per = (m + 3) / 4, g = tid >> 8, t = tid & 255;
    const int c0 = g * per, mine = m - c0 < per ? m - c0 : per;   // candidates of this group (may be <= 0)
    float acc[RG];
#pragma unroll
    for (int j = 0; j < RG; ++j) acc[j] = 0.f;
    if (mine > 0) {
        for (int64_t i = (int64_t)t * 8; i < a.d; i += 256 * 8) {
            const f32x4 q0 = *reinterpret_cast<const f32x4 *>(qrow + i);
            const f32x4 q1 = *reinterpret_cast<const f32x4 *>(qrow + i + 4);
            const float qv[8] = {q0[0], q0[1], q0[2], q0[3], q1[0], q1[1], q1[2], q1[3]};
            if (a.c_f32) {
#pragma unroll
                for (int j = 0; j < RG; ++j) {
                    const float *c = a.c_f32 + (int64_t)idx_s[c0 + (j < mine ? j : mine - 1)] * a.d_pad + i;
                    const f32x4 c0v = *reinterpret_cast<const f32x4 *>(c);
                    const f32x4 c1v = *reinterpret_cast<const f32x4 *>(c + 4);
                    const float cv[8] = {c0v[0], c0v[1], c0v[2], c0v[3], c1v[0], c1v[1], c1v[2], c1v[3]};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float df = qv[e] - cv[e];
                        acc[j] = __builtin_fmaf(df, df, acc[j]);
                    }
                }
            } else {
                uint4 cb[RG];
#pragma unroll
                for (int j = 0; j < RG; ++j)
                    cb[j] = *reinterpret_cast<const uint4 *>(a.c_rows + (int64_t)idx_s[c0 + (j < mine ? j : mine - 1)] * a.d_pad + i);
#pragma unroll
                for (int j = 0; j < RG; ++j) {
                    const uint32_t wv[4] = {cb[j].x, cb[j].y, cb[j].z, cb[j].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float d0 = qv[2 * e] - __uint_as_float(wv[e] << 16);
                        acc[j] = __builtin_fmaf(d0, d0, acc[j]);
                        const float d1 = qv[2 * e + 1] - __uint_as_float(wv[e] & 0xffff0000u);
                        acc[j] = __builtin_fmaf(d1, d1, acc[j]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < RG; ++j) {
        float v = acc[j];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((tid & 63) == 0) red[tid >> 6][j] = v;
    }
    __syncthreads();
    if (t < RG && t < mine)
        dist_s[c0 + t] = 0.f + ((red[4 * g][t] + red[4 * g + 1][t]) + (red[4 * g + 2][t] + red[4 * g + 3][t]));
    __syncthreads();
}

__global__ __launch_bounds__(kThrThreads) void keys_finish_kernel(KeysFinishArgs ka)
{
    const FinishArgs &a = ka.a;
    __shared__ uint64_t list[kThrList];          // gathered minima, then the candidates
    __shared__ uint64_t pick_s[kMaxRescore];     // minima of the selected blocks
    __shared__ uint64_t grp_s[kThrGroups];
    __shared__ int rank_s[kThrGroups];
    __shared__ uint64_t sel_s;
    __shared__ int list_n, blk_n, cand_n, distinct_s, verdict_s, last_s;
    __shared__ float red16[16][16];
    __shared__ float dist_s[kMaxRescore];
    __shared__ int32_t idx_s[kMaxRescore];
    __shared__ int32_t lab_s[kMaxK], cnt_s[kMaxK];
    __shared__ float dsel_s[kMaxK];
    __shared__ double conf_s[kMaxK];
    __shared__ int32_t nearest_s;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (a.count && q >= *a.count) return;   // uniform
    const int64_t nb = ka.nb;
    const int r = a.r, r_sel = ka.r_sel;
    const uint64_t *bq = ka.bmin + (size_t)q * nb;

    // ---- 1. blocks that can hold a candidate ----
    if (tid == 0) {
        list_n = 0;
        blk_n = 0;
        cand_n = 0;
        distinct_s = 0;
    }
    if (tid < kThrGroups) rank_s[tid] = 0;
    uint64_t t = kSentinel;   // threshold on (key, index) pairs
    const float *kq = ka.keys + (size_t)q * ka.n_pad;
    const bool by_entry = r_sel >= nb;   // as few blocks as that: groups of entries in their place
    int nblk = 0;
    {
        constexpr int NV = 8;   // minima per thread kept in registers
        static_assert(kMaxRescore * 32 <= NV * kThrThreads, "all entries by entry");
        const int64_t values = by_entry ? a.n : nb;
        uint64_t v[NV], m = kSentinel;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int64_t j = (int64_t)i * kThrThreads + tid;
            v[i] = kSentinel;
            if (j < values) v[i] = by_entry ? ((uint64_t)ordered_bits(kq[j]) << 32) | (uint32_t)j : bq[j];
            m = v[i] < m ? v[i] : m;
        }
        for (int64_t j = (int64_t)NV * kThrThreads + tid; j < nb; j += kThrThreads) {
            const uint64_t x = bq[j];
            m = x < m ? x : m;
        }
        list[tid] = m;
        __syncthreads();
        if (tid < kThrGroups) {
            uint64_t g = list[tid];
#pragma unroll
            for (int i = 1; i < kThrThreads / kThrGroups; ++i) {
                const uint64_t x = list[tid + i * kThrGroups];
                g = x < g ? x : g;
            }
            grp_s[tid] = g;
        }
        __syncthreads();
        {   // rank of every group minimum: four threads count a quarter of the others each
            const uint64_t mine = grp_s[tid & (kThrGroups - 1)];
            const int part = tid / kThrGroups * (kThrGroups / 4);
            int c = 0;
#pragma unroll 16
            for (int j = 0; j < kThrGroups / 4; ++j) c += grp_s[part + j] < mine;
            atomicAdd(&rank_s[tid & (kThrGroups - 1)], c);
        }
        __syncthreads();
        // (groups without a value hold the marker; where the values lie in fewer than r_sel groups T stays the marker and
        // everything passes)
        if (tid == 0) sel_s = kSentinel;
        __syncthreads();
        if (tid < kThrGroups && rank_s[tid] == r_sel - 1 && grp_s[tid] != kSentinel) sel_s = grp_s[tid];
        __syncthreads();
        t = sel_s;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (v[i] <= t && v[i] != kSentinel) {
                const int pos = atomicAdd(&list_n, 1);
                if (pos < kThrList) list[pos] = v[i];
            }
        }
        for (int64_t j = (int64_t)NV * kThrThreads + tid; j < nb; j += kThrThreads) {
            const uint64_t x = bq[j];
            if (x <= t) {
                const int pos = atomicAdd(&list_n, 1);
                if (pos < kThrList) list[pos] = x;
            }
        }
        __syncthreads();
        const int cnt = list_n < kThrList ? list_n : kThrList;
        if (by_entry) {   // uniform
            if (tid == 0) cand_n = cnt;
        } else if (cnt <= kMaxRescore) {
            if (tid < cnt) pick_s[tid] = list[tid];
            nblk = cnt;
        } else {   // uniform
            t = rth_of_list(list, cnt, r_sel, &sel_s, tid);
            __syncthreads();
            for (int i = tid; i < cnt; i += kThrThreads) {
                const uint64_t x = list[i];
                if (x <= t) {
                    const int pos = atomicAdd(&blk_n, 1);
                    if (pos < kMaxRescore) pick_s[pos] = x;
                }
            }
            nblk = r_sel;
        }
        __syncthreads();
    }

    // ---- their entries at or under the threshold, in order of their keys ----
    for (int c = tid; c < nblk * 32; c += kThrThreads) {
        const uint32_t idx = ((uint32_t)pick_s[c >> 5] & ~31u) + (c & 31);
        const uint64_t pr = ((uint64_t)ordered_bits(kq[idx]) << 32) | idx;
        if (pr <= t && idx < (uint32_t)a.n) list[atomicAdd(&cand_n, 1)] = pr;   // <= 64 * 32 entries
    }
    __syncthreads();
    const int real = cand_n;
    int have = real;
    if (have <= 64) {
        if (w == 0) list[lane] = wave_sort64(lane < have ? list[lane] : kSentinel, lane);
        __syncthreads();
    } else {
        int n2 = 128;
        while (n2 < have) n2 <<= 1;
        for (int i = have + tid; i < n2; i += kThrThreads) list[i] = kSentinel;
        __syncthreads();
        bitonic_sort_lds(list, n2, tid, kThrThreads);
    }

    // ---- 2. exact re-scoring of the first r ----
    if (tid < r) {
        // (fewer than r candidates, i.e. markers here, only with non-finite inputs: mapped to row 0)
        const uint32_t ci = (uint32_t)list[tid];
        idx_s[tid] = ci < (uint32_t)a.n ? (int32_t)ci : 0;
    }
    __syncthreads();
    const float *qrow = a.queries + (int64_t)(a.sel ? a.sel[q] : q) * a.d;
    auto rescore = [&](int c0, int m) {
        if (a.d >= 16384 && a.d % 8 == 0) {
            float(*red)[8] = reinterpret_cast<float(*)[8]>(&red16[0][0]);
            if (m <= 2) {
                rescore_block_all<1024, 2, false, 2>(a, qrow, idx_s + c0, dist_s + c0, red, m, tid);
            } else if (m <= 4) {
                rescore_block_all<1024, 4, false, 4>(a, qrow, idx_s + c0, dist_s + c0, red, m, tid);
            } else if (m <= 16) {
                rescore_block_all<1024, 16>(a, qrow, idx_s + c0, dist_s + c0, red, m, tid);
            } else {
                for (int c = 0; c < m; c += 32)
                    rescore_block_all<1024, 32>(a, qrow, idx_s + c0 + c, dist_s + c0 + c, red, m - c < 32 ? m - c : 32, tid);
            }
        } else if (a.d >= 4096 && a.d % 8 == 0) {
            if (m <= 4)
                rescore_groups<1>(a, qrow, idx_s + c0, dist_s + c0, reinterpret_cast<float(*)[1]>(&red16[0][0]), m, tid);
            else if (m <= 16)
                rescore_groups<4>(a, qrow, idx_s + c0, dist_s + c0, reinterpret_cast<float(*)[4]>(&red16[0][0]), m, tid);
            else if (m <= 32)
                rescore_groups<8>(a, qrow, idx_s + c0, dist_s + c0, reinterpret_cast<float(*)[8]>(&red16[0][0]), m, tid);
            else
                rescore_groups<16>(a, qrow, idx_s + c0, dist_s + c0, red16, m, tid);
        } else {
            if (m <= 16)
                rescore_wave<1>(a, qrow, idx_s + c0, dist_s + c0, m, w, lane, 16);
            else if (m <= 32)
                rescore_wave<2>(a, qrow, idx_s + c0, dist_s + c0, m, w, lane, 16);
            else
                rescore_wave<4>(a, qrow, idx_s + c0, dist_s + c0, m, w, lane, 16);
        }
        __syncthreads();
    };
    const int m_first = ka.m_first;
    if (ka.parts > 1) {   // uniform
        const int per = (m_first + ka.parts - 1) / ka.parts, c0 = (int)blockIdx.y * per, m = m_first - c0 < per ? m_first - c0 : per;
        if (m > 0) rescore(c0, m);   // uniform
        // (device-coherent stores, complete before the ticket is taken, and device-coherent loads: as in follow_up_kernel)
        float *meet = ka.meet + (size_t)q * kMaxRescore;
        if (tid >= c0 && tid < c0 + m) __hip_atomic_store(meet + tid, dist_s[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) {
            last_s = atomicAdd(&ka.tickets[q], 1) == ka.parts - 1;
            if (last_s) atomicExch(&ka.tickets[q], 0);   // the exact scan's tickets are these
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(last_s)) return;   // uniform: the query's last workgroup goes on
        if (tid < m_first) dist_s[tid] = __hip_atomic_load(meet + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    } else {
        rescore(0, m_first);
    }

    // ---- 3. final order, certificate, vote ----
    // every entry that is no candidate has a key at or above the largest candidate's
    const uint32_t excl0 = real >= a.n || real < 1 ? 0xffffffffu : (uint32_t)(list[real - 1] >> 32);
    auto confirm = [&](int m) {
        rank_and_emit(a, q, m, tid, kThrThreads, dist_s, idx_s, lab_s, dsel_s, &nearest_s, &distinct_s);
        __syncthreads();
        uint32_t excl = excl0;
        if (real > m) {
            const uint32_t nxt = (uint32_t)(list[m] >> 32);
            excl = nxt < excl ? nxt : excl;
        }
        return __builtin_amdgcn_readfirstlane((int)certificate(list, dist_s, m, dsel_s[a.k - 1], excl, distinct_s, tid, &verdict_s)) != 0;
    };
    bool ok = confirm(m_first);
    if (!ok && m_first < r) {   // uniform
        rescore(m_first, r - m_first);
        if (tid == 0) distinct_s = 0;
        __syncthreads();
        ok = confirm(r);
    }
    if (__builtin_expect(!ok, 0)) {   // uniform (and out of the way of the instruction fetch)
        // Unconfirmed: the wider re-scoring, or the exact scan, redoes this query.  The candidates at hand do when
        // their largest key as the bound would have confirmed the result.  Else (duplicates, neighbours closer than
        // the key's error) the wider re-scoring gets at least the kTier1 entries with the smallest keys: T2 = the largest
        // of the sixteen waves' sixteenth smallest thread minima, over entries on small caches, over blocks on others.
        // (50,000 x 8,192, 32 queries, 21 copies of every entry: 2,484 us by the exact scan, 275 so.)
        const uint64_t *src = list;
        int keep = real;
        __syncthreads();   // (everyone has read the verdict that this one replaces)
        const bool enough = certificate(list, dist_s, r, dsel_s[a.k - 1], excl0, distinct_s, tid, &verdict_s);
        if (!enough && real < kTier1 && real < a.n) {   // uniform
            uint64_t *wide = list + kThrList / 2;   // (the candidates at hand stay in the first 2,048 places)
            const bool by_entry = nb < kThrThreads;
            auto entry = [&](int64_t i) { return ((uint64_t)ordered_bits(kq[i]) << 32) | (uint32_t)i; };
            uint64_t m = kSentinel;
            for (int64_t j = tid; j < (by_entry ? a.n : nb); j += kThrThreads) {
                const uint64_t x = by_entry ? entry(j) : bq[j];
                m = x < m ? x : m;
            }
            const uint64_t c = wave_sort64(m, lane);
            static_assert(kTier1 / (kThrThreads / 64) == 16, "sixteen per wave");
            if (lane == 15) grp_s[w] = c;
            if (tid == 0) cand_n = 0;
            __syncthreads();
            uint64_t t2 = grp_s[0];
#pragma unroll
            for (int i = 1; i < kThrThreads / 64; ++i) t2 = grp_s[i] > t2 ? grp_s[i] : t2;
            auto take = [&](uint64_t pr) {
                const int pos = atomicAdd(&cand_n, 1);
                if (pos < kThrList / 2) wide[pos] = pr;
            };
            for (int64_t j = tid; j < (by_entry ? a.n : nb); j += kThrThreads) {
                const uint64_t x = by_entry ? entry(j) : bq[j];
                if (x <= t2) {
                    if (by_entry) {
                        take(x);
                    } else {
                        const uint32_t i0 = (uint32_t)x & ~31u;
                        for (uint32_t i = i0; i < i0 + 32; i += 4) {
                            const f32x4 v = *reinterpret_cast<const f32x4 *>(kq + i);
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const uint64_t pr = ((uint64_t)ordered_bits(v[e]) << 32) | (i + e);
                                if (pr <= t2 && i + e < (uint32_t)a.n) take(pr);
                            }
                        }
                    }
                }
            }
            __syncthreads();
            const int got = cand_n;
            if (got <= kThrList / 2 && got > real) {   // uniform (more than fit: the candidates at hand are handed on)
                if (got > a.part_stride) {   // (the wider re-scoring sorts what it gets; here only what is cut off must be the largest)
                    int n2 = 64;
                    while (n2 < got) n2 <<= 1;
                    for (int i = got + tid; i < n2; i += kThrThreads) wide[i] = kSentinel;
                    __syncthreads();
                    bitonic_sort_lds(wide, n2, tid, kThrThreads);
                }
                src = wide;
                keep = got;
            }
        }
        keep = keep < a.part_stride ? keep : a.part_stride;
        for (int i = tid; i < keep; i += kThrThreads) ka.cand[(size_t)q * a.part_stride + i] = src[i];
        if (tid == 0) {
            ka.cand_count[q] = keep;
            const int next = keep <= r ? 1 : 0;
            const int pos = atomicAdd(a.flag_count + next, 1);
            (next ? a.flag_list2 : a.flag_list)[pos] = q;
            if (a.stats && next == 1) atomicAdd(a.stats + 2, 1ull);
        }
    } else if (tid == 0 && a.stats) {
        atomicAdd(a.stats, 1ull);
    }
    decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
}

bool keys_finish_supported(int64_t n_pad, int r)
{
    const int64_t nb = n_pad / 32;
    return ((nb + kThrGroups - 1) / kThrGroups) * r <= kThrList;
}

int keys_finish_cand(int r) { return 32 * r < 2 * kTier1 ? 32 * r : 2 * kTier1; }

size_t keys_finish_meet_entries(int64_t rows) { return rows <= kPartsRows ? (size_t)rows * kMaxRescore : 0; }

size_t keys_finish_workspace_bytes(int64_t rows, int64_t n_pad, int r, size_t align)
{
    auto up = [&](size_t x) { return (x + align - 1) / align * align; };
    const size_t b = (size_t)rows;
    return up(b * (size_t)n_pad * 4) + up(b * (size_t)(n_pad / 32) * 8) + up(b * 4) + up(b * (size_t)keys_finish_cand(r) * 8);
}

// a.part / a.part_count (stride keys_finish_cand(a.r)) are the kernel's outputs for the wider re-scoring
hipError_t launch_keys_finish(const FinishArgs &a, const float *keys, const uint64_t *bmin, int64_t n_pad, uint64_t *cand,
                              int32_t *cand_count, float *meet, int32_t *tickets, int num_cus, hipStream_t s)
{
    if (!keys_finish_supported(n_pad, a.r) || a.r < 1 || a.r > kMaxRescore || a.k > kMaxK || a.k > a.r || a.b < 1 || !a.flag_count ||
        !a.flag_list || !a.flag_list2 || a.part_stride != keys_finish_cand(a.r))
        return hipErrorInvalidValue;
    const int64_t nb = n_pad / 32, per_group = (nb + kThrGroups - 1) / kThrGroups;
    int r_sel = 2 * a.r < kMaxRescore ? 2 * a.r : kMaxRescore;
    // Not more than half of few blocks where that leaves the width: the threshold is the r_sel-th smallest block minimum, and near
    // the largest it lets in a good part of the cache, which is sorted.  One query, 2,000 x 512 (64 blocks), k = 20: 41 us with
    // all blocks, 26 with half of them; k = 40, by entries, 45 -> 33.
    if (r_sel > nb / 2) r_sel = a.r > nb / 2 ? a.r : (int)(nb / 2);
    while (r_sel > a.r && per_group * r_sel > kThrList) --r_sel;   // the gathered minima fit the list
    KeysFinishArgs ka{a, bmin, keys, nb, n_pad, r_sel, cand, cand_count, first_width(a, a.b > 64), 1, meet, tickets};
    // Long rows, few queries: a workgroup gets a row out of memory at 50 to 100 GB/s, so up to eight share the rows of a query,
    // 32 KB each at least; each repeats the selection.  One query,
    // 50,000 x 16,384: 22 -> 16 us of this kernel; 4 x 3,404 x 16,384 fp32, k = 20: 52 -> 21; 60 x 3,433 x 16,384, k = 20: 40 -> 28; 32 x
    // 50,000 x 65,536 .. 16,384: 32 -> 17.
    if (meet && tickets && a.d >= 4096) {
        const int64_t bytes = (int64_t)ka.m_first * a.d_pad * (a.c_f32 ? 4 : 2);
        int64_t parts = bytes / 32768;
        parts = parts < num_cus / a.b ? parts : num_cus / a.b;
        parts = parts < 8 ? parts : 8;
        if (parts > 1) {
            const int per = (int)((ka.m_first + parts - 1) / parts);
            ka.parts = (ka.m_first + per - 1) / per;
        }
    }
    hipLaunchKernelGGL(keys_finish_kernel, dim3((unsigned)a.b, (unsigned)ka.parts), dim3(kThrThreads), 0, s, ka);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Finishing kernel of the block-minima route, one workgroup of 128 or
// 256 threads per query, from the smallest coarse key of every block of eight entries:
//  1. Selection.  Every wave takes the (2 R / waves)-th smallest of its 64 lanes' minima; T = the largest of
//     these.  At least 2 R block minima are <= T, usually a few more: those are gathered and sorted.  The
//     first m of them hold the m best entries by the coarse key: each holds one that is no worse than any
//     entry outside them.
//  2. Exact re-scoring, of the first k + 2 blocks at first: of each the entry that has the smallest key, where the
//     matrix kernel has left that (NEXT), and all eight where the bound of the others' keys lies under the smallest key that is
//     left out (two of the nearest in one block; no lead, i.e. equal keys).  Without it, all eight of every block.  Eight rows
//     in flight per lane, and one transposed reduction for the eight sums (ten shuffles instead of 48).  Same order of
//     additions as in the other kernels (rescore_rows8), hence the same distances bit for bit.
//  3. The k nearest by (distance, index).
//  4. The certificate.  Its samples are the blocks' smallest keys and the distances of the entries that have them (NEXT).
//     Without NEXT it is not known which that is: the coarse key of
//     the block's nearest entry is formed again from the same bf16 values (the query's and the row's,
//     relative to the cache's mean where the matrix cores' copy is), and what this sample does not show, the rounding of the
//     matrix cores' additions, at most one ulp of a partial sum per k-step, the margin's floor covers.
//     Entries outside the blocks taken have a key at or above the next minimum, and so have those that were passed over in
//     them.  A query that fails takes R blocks, then all that were gathered (up to 64), then up to 256.
//  5. The 256 are selected anew and re-scored like the first ones.  The first kMeetQueries queries that get here leave that to the
//     follow-up kernel, where sixteen workgroups share each: that is all of them on most inputs, and a single workgroup would
//     be the last to finish by far.  With more (duplicates, neighbours closer than the key's error) the chip is busy
//     anyway, and each goes on here.
// Bound by its chain of dependent steps and the minima it reads (103 MB at 4,096 queries x 50,000): 70 - 76 us for 4,096
// queries x 50,000 x 512, k = 10, with NEXT; 137 - 155 with eight rows per block, 0.4 GB and more beyond L2 (51 MB of cache).
// ---------------------------------------------------------------------------------------
constexpr int kMeetQueries = 32;
struct BlockFinishArgs {
    FinishArgs a;
    const float *bkey;   // [b, nb] smallest coarse key of every block
    const uint16_t *bnext;   // [b, nb] which entry has it, and a bound of the others (block_others)
    const float *norm;   // [n_pad]
    const float *mu;     // [d_pad] centring vector or null
    int64_t nb;
    int64_t real_blocks; // blocks that hold an entry (the others hold padding rows)
    int nk;              // k-steps of the matrix-core pass
    int first;           // blocks re-scored at first
    int gather;          // blocks the threshold lets in at least
};

// first of the eight entries of block blk: entries first + e and first + 16 + e, e < 4
__host__ __device__ inline int block_first_entry(int blk)
{
    return (blk >> 5) * kTileN + ((blk >> 3) & 3) * 64 + (blk & 1) * 32 + ((blk >> 1) & 3) * 4;
}

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
// two values rounded to bf16 (nearest even) and widened again
__device__ __forceinline__ f32x2 through_bf16(float x, float y)
{
    const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
    return f32x2{__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u)};
}

// the query's elements i .. i + 7 (zeros past d, where the cache's rows are zero too)
__device__ __forceinline__ void load_query8(const float *qrow, int64_t i, int64_t d, float (&x)[8])
{
    if ((d % 8) == 0 || ((d % 4) == 0 && i + 8 <= d)) {   // 16-byte aligned
        const f32x4 q0 = *reinterpret_cast<const f32x4 *>(qrow + i), q1 = *reinterpret_cast<const f32x4 *>(qrow + i + 4);
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = e < 4 ? q0[e & 3] : q1[e & 3];
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = i + e < d ? qrow[i + e] : 0.f;
    }
}

// The eight entries of the block that starts at entry e0 (uniform).
struct BlockRows {
    int e0;
    __device__ __forceinline__ int operator()(int j) const { return e0 + (j & 3) + (j >> 2) * 16; }
    __device__ __forceinline__ int uniform(int j) const { return (*this)(j); }
};

// Eight entries anywhere: of(j), the same in every lane, and first[j] = of(j) in scalar registers.
template <class F>
struct ListRows {
    const F &of;
    int first[8];
    __device__ __forceinline__ int operator()(int j) const { return of(j); }
    __device__ __forceinline__ int uniform(int j) const { return first[j]; }
};

// Exact distances of the eight entries rows(0 .. 7), by one wave: the packed (distance, index) of row lane >> 3 in every
// lane, the marker where that is no entry.  Same order of additions as in the other kernels for rows of any length (the
// longest of few queries, wide_order, do not come here): rescore_block_all<256, .>'s four waves' chains, one after the other,
// from 4,096 on, rescore_wave's else.
template <class Rows>
__device__ __forceinline__ uint64_t rescore_rows8(const FinishArgs &a, const float *qrow, const Rows &rows, int lane)
{
    const bool whole = (a.d % 8) == 0;
    // the row's place in the cache (uniform); rows past it (padding) are read as the last row and dropped below
    auto row_of = [&](int j) {
        const int e = rows.uniform(j);
        return (int64_t)((uint32_t)e < (uint32_t)a.n ? e : a.n - 1) * a.d_pad;
    };
    float acc[8];
    // transposed reduction: after the steps over lane bits 5, 4 and 3 a lane holds the partial sum of
    // row 4 b5 + 2 b4 + b3, the rest is a butterfly
    auto reduce = [&]() {
        float s4[4], s2[2], s1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const bool hi = lane & 32;
            s4[j] = (hi ? acc[4 + j] : acc[j]) + __shfl_xor(hi ? acc[j] : acc[4 + j], 32, 64);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const bool hi = lane & 16;
            s2[j] = (hi ? s4[2 + j] : s4[j]) + __shfl_xor(hi ? s4[j] : s4[2 + j], 16, 64);
        }
        {
            const bool hi = lane & 8;
            s1 = (hi ? s2[1] : s2[0]) + __shfl_xor(hi ? s2[0] : s2[1], 8, 64);
        }
#pragma unroll
        for (int off = 4; off >= 1; off >>= 1) s1 += __shfl_xor(s1, off, 64);
        return s1;
    };
    float s1;
    if (whole) {   // uniform
        const int chains = a.d >= 4096 ? 4 : 1;
        float pair = 0.f;
        s1 = 0.f;
        for (int c = 0; c < chains; ++c) {
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = 0.f;
            for (int64_t i = (int64_t)(c * 64 + lane) * 8; i < a.d; i += 512 * chains) {
                float qv[8];
                load_query8(qrow, i, a.d, qv);
                if (a.c_f32) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const f32x4 c0 = *reinterpret_cast<const f32x4 *>(a.c_f32 + row_of(j) + i);
                        const f32x4 c1 = *reinterpret_cast<const f32x4 *>(a.c_f32 + row_of(j) + i + 4);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float df = qv[e] - (e < 4 ? c0[e & 3] : c1[e & 3]);
                            acc[j] = __builtin_fmaf(df, df, acc[j]);
                        }
                    }
                } else {
                    uint4 cb[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) cb[j] = *reinterpret_cast<const uint4 *>(a.c_rows + row_of(j) + i);
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t wv[4] = {cb[j].x, cb[j].y, cb[j].z, cb[j].w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float d0 = qv[2 * e] - __uint_as_float(wv[e] << 16);
                            acc[j] = __builtin_fmaf(d0, d0, acc[j]);
                            const float d1 = qv[2 * e + 1] - __uint_as_float(wv[e] & 0xffff0000u);
                            acc[j] = __builtin_fmaf(d1, d1, acc[j]);
                        }
                    }
                }
            }
            // one chain: its sum; four: (0 + 1) + (2 + 3)
            const float sum = reduce();
            if (c & 1) s1 += pair + sum;
            else pair = sum;
        }
        if (chains == 1) s1 = pair;
    } else if (a.c_f32) {
        // Rows of another length: rescore_wave's order, chain l of 64 takes elements l, l + 64, .., so that a
        // distance does not depend on the kernel that formed it.  A chain per lane; four steps' loads of all
        // eight rows in flight (whole look-ups, 20,011 x 517, 1,537 queries, k = 20: 242 us with eight elements per lane, 189 so).
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.f;
        auto steps = [&](int64_t i, auto count) {
            constexpr int U = decltype(count)::value;
            float qv[U], cv[8][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                qv[u] = qrow[i + u * 64];
#pragma unroll
                for (int j = 0; j < 8; ++j) cv[j][u] = a.c_f32[row_of(j) + i + u * 64];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const float df = qv[u] - cv[j][u];
                    acc[j] = __builtin_fmaf(df, df, acc[j]);
                }
        };
        int64_t i = lane;
        for (; i + 3 * 64 < a.d; i += 4 * 64) steps(i, std::integral_constant<int, 4>{});
        for (; i < a.d; i += 64) steps(i, std::integral_constant<int, 1>{});
        s1 = reduce();
    } else {
        // The same order on bf16 rows: half a wave per row, chains 2 p and 2 p + 1 in lane p of the half, so that a
        // lane's load is 4 bytes (50,000 x 517, 4,096 queries: 363 us with eight elements per lane, 708 with a chain per lane
        // and 2-byte loads, 350 so).  Lane bit 5 and jp name the row; elements past d are zeros on both sides and
        // leave a chain as it is.
        const int p = lane & 31, hf = lane >> 5;
        const uint32_t *row[4];
#pragma unroll
        for (int jp = 0; jp < 4; ++jp) {
            const int e = rows(jp + hf * 4);
            row[jp] = reinterpret_cast<const uint32_t *>(a.c_rows + (int64_t)((uint32_t)e < (uint32_t)a.n ? e : a.n - 1) * a.d_pad) + p;
        }
        float ch[4][2];   // [jp][chain of the lane]
#pragma unroll
        for (int jp = 0; jp < 4; ++jp) ch[jp][0] = ch[jp][1] = 0.f;
        auto steps = [&](int64_t i0, auto count) {   // elements [i0, i0 + 64 U), i0 + 64 U <= d_pad
            constexpr int U = decltype(count)::value;
            float qv[U][2];
            uint32_t cv[4][U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + u * 64 + 2 * p;
#pragma unroll
                for (int h = 0; h < 2; ++h) qv[u][h] = i + h < a.d ? qrow[i + h] : 0.f;
#pragma unroll
                for (int jp = 0; jp < 4; ++jp) cv[jp][u] = row[jp][(i0 >> 1) + u * 32];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int jp = 0; jp < 4; ++jp) {
                    const float d0 = qv[u][0] - __uint_as_float(cv[jp][u] << 16);
                    ch[jp][0] = __builtin_fmaf(d0, d0, ch[jp][0]);
                    const float d1 = qv[u][1] - __uint_as_float(cv[jp][u] & 0xffff0000u);
                    ch[jp][1] = __builtin_fmaf(d1, d1, ch[jp][1]);
                }
        };
        int64_t i0 = 0;
        for (; i0 + 4 * 64 <= a.d_pad; i0 += 4 * 64) steps(i0, std::integral_constant<int, 4>{});
        for (; i0 < a.d_pad; i0 += 64) steps(i0, std::integral_constant<int, 1>{});
        // the butterfly over chains 32, 16, 8, 4, 2 and 1 apart: lanes 16, 8, 4, 2 and 1 apart, then the
        // lane's two chains; transposed over lane bits 4 and 3 (jp) and 2 (the chain)
        float t4[2][2], t2[2];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const bool hi = lane & 16;
                t4[j][h] = (hi ? ch[2 + j][h] : ch[j][h]) + __shfl_xor(hi ? ch[j][h] : ch[2 + j][h], 16, 64);
            }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bool hi = lane & 8;
            t2[h] = (hi ? t4[1][h] : t4[0][h]) + __shfl_xor(hi ? t4[0][h] : t4[1][h], 8, 64);
        }
        {
            const bool hi = lane & 4;
            s1 = (hi ? t2[1] : t2[0]) + __shfl_xor(hi ? t2[0] : t2[1], 4, 64);
        }
        s1 += __shfl_xor(s1, 2, 64);
        s1 += __shfl_xor(s1, 1, 64);
        s1 += __shfl_xor(s1, 4, 64);
    }
    // lane >> 3 = 4 b5 + 2 b4 + b3: the row
    const int e = rows(lane >> 3);
    return (uint32_t)e < (uint32_t)a.n ? ((uint64_t)ordered_bits(s1) << 32) | (uint32_t)e : kSentinel;
}

// The smallest of the eight rows' values of rescore_rows8.
__device__ __forceinline__ uint64_t block_nearest(uint64_t x)
{
#pragma unroll
    for (int off = 32; off >= 8; off >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)x, off, 64);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(x >> 32), off, 64);
        const uint64_t y = ((uint64_t)hi << 32) | lo;
        x = y < x ? y : x;
    }
    return x;
}

// Dot products of the bf16 copies of the query and of entries idx[b0 .. b0 + 3] (of m), as the coarse keys are made of,
// relative to mu where that is given, by one wave: that of entry b0 + (lane >> 4) in every lane.
__device__ __forceinline__ float coarse_dot4(const FinishArgs &a, const float *mu, const float *qrow, const int32_t *idx, int b0, int m, int lane)
{
    int64_t row[4];
    float dot[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        row[j] = (int64_t)__builtin_amdgcn_readfirstlane(idx[b0 + j < m ? b0 + j : m - 1]) * a.d_pad;
        dot[j] = 0.f;
    }
    for (int64_t i = (int64_t)lane * 8; i < a.d; i += 512) {
        float qv[8], mv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        load_query8(qrow, i, a.d, qv);
        if (mu) {
            const f32x4 m0 = *reinterpret_cast<const f32x4 *>(mu + i), m1 = *reinterpret_cast<const f32x4 *>(mu + i + 4);
#pragma unroll
            for (int e = 0; e < 8; ++e) mv[e] = e < 4 ? m0[e & 3] : m1[e & 3];
        }
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const f32x2 v = through_bf16(qv[e] - mv[e], qv[e + 1] - mv[e + 1]);
            qv[e] = v[0];
            qv[e + 1] = v[1];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float cv[8];
            if (a.c_f32) {
                const f32x4 c0 = *reinterpret_cast<const f32x4 *>(a.c_f32 + row[j] + i);
                const f32x4 c1 = *reinterpret_cast<const f32x4 *>(a.c_f32 + row[j] + i + 4);
#pragma unroll
                for (int e = 0; e < 8; ++e) cv[e] = e < 4 ? c0[e & 3] : c1[e & 3];
            } else {
                const uint4 cb = *reinterpret_cast<const uint4 *>(a.c_rows + row[j] + i);
                const uint32_t wv[4] = {cb.x, cb.y, cb.z, cb.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    cv[2 * e] = __uint_as_float(wv[e] << 16);
                    cv[2 * e + 1] = __uint_as_float(wv[e] & 0xffff0000u);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const f32x2 v = through_bf16(cv[e] - mv[e], cv[e + 1] - mv[e + 1]);
                dot[j] = __builtin_fmaf(qv[e], v[0], dot[j]);
                dot[j] = __builtin_fmaf(qv[e + 1], v[1], dot[j]);
            }
        }
    }
    // the four sums, transposed: lane bits 5 and 4 name the row
    float s2[2], s1;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const bool hi = lane & 32;
        s2[j] = (hi ? dot[2 + j] : dot[j]) + __shfl_xor(hi ? dot[j] : dot[2 + j], 32, 64);
    }
    {
        const bool hi = lane & 16;
        s1 = (hi ? s2[1] : s2[0]) + __shfl_xor(hi ? s2[0] : s2[1], 16, 64);
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) s1 += __shfl_xor(s1, off, 64);
    return s1;
}

// NEXT: of a block it is known which entry has the smallest key, and a bound of the others'; else all eight are re-scored.
template <int NT, bool NEXT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(4))) void block_finish_kernel(BlockFinishArgs ba)
{
    const FinishArgs &a = ba.a;
    constexpr int NW = NT / 64;
    constexpr int RMAX = kMaxRescore;                 // blocks taken before the 256 at most
    constexpr int kBlkList = 4 * NT;                  // gathered minima at most
    __shared__ uint64_t list[kBlkList];
    __shared__ uint64_t ent[RMAX * 16];               // entries of the blocks; group minima
    uint64_t *ent2 = ent + RMAX * 8;
    static_assert(RMAX * 16 >= kBlkList && kBlkList >= 2 * kTier1, "step 5");
    __shared__ uint64_t samp_s[kTier1];
    __shared__ float sdist_s[kTier1];
    __shared__ int32_t sidx_s[kTier1];
    __shared__ uint64_t best_s[kMaxK];
    __shared__ uint32_t wave_s[4];
    __shared__ int32_t lab_s[kMaxK], cnt_s[kMaxK];
    __shared__ float dsel_s[kMaxK];
    __shared__ double conf_s[kMaxK];
    __shared__ int32_t nearest_s;
    __shared__ uint64_t kth_s;
    __shared__ int list_n, near_n, open_n, distinct_s, verdict_s, flagged_s;
    __shared__ float others_s[RMAX];                  // bound of the keys of a block's other entries; +inf: they have been re-scored, too
    __shared__ uint8_t at_s[kTier1];                  // which of a block's entries has the smallest key; step 5: 8 more, all of them
    __shared__ uint16_t work_s[RMAX * 8];             // slots to re-score
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (a.count && q >= *a.count) return;   // uniform
    const int r = a.r;
    const float *bq = ba.bkey + (size_t)q * ba.nb;
    constexpr uint32_t kInf = 0xff800000u;   // ordered bits of +inf: a block of padding rows, or no block
    const float inf = __builtin_inff();

    // ---- 1. selection ----
    if (tid == 0) list_n = 0;
    uint32_t t1;
    {
        // group j of a thread: four consecutive minima, or with few blocks a single one, so that every lane has some
        const bool by_four = ba.nb > 8 * NT;
        const int64_t ng = by_four ? ba.nb / 4 : ba.nb;
        auto fetch = [&](int64_t j) {
            if (by_four) return reinterpret_cast<const f32x4 *>(bq)[j];
            return f32x4{bq[j], inf, inf, inf};
        };
        // the minimum of every group; those of a thread's first G groups stay in registers, so that the second
        // look fetches the few groups that hold something (further ones are read again: caches of more than
        // 65,536 entries)
        constexpr int G = 2048 / NT, U = 8;   // U groups in flight
        float gm[G], m = inf;
        auto group_min = [&](int64_t j) {
            const f32x4 v = j < ng ? fetch(j) : f32x4{inf, inf, inf, inf};
            return __builtin_fminf(__builtin_fminf(v[0], v[1]), __builtin_fminf(v[2], v[3]));
        };
#pragma unroll
        for (int i0 = 0; i0 < G; i0 += U) {
#pragma unroll
            for (int i = i0; i < i0 + U; ++i) gm[i] = group_min((int64_t)i * NT + tid);
        }
#pragma unroll
        for (int i = 0; i < G; ++i) m = __builtin_fminf(m, gm[i]);
        for (int64_t j0 = (int64_t)G * NT + tid; j0 < ng; j0 += (int64_t)U * NT) {
            float t[U];
#pragma unroll
            for (int i = 0; i < U; ++i) t[i] = group_min(j0 + (int64_t)i * NT);
#pragma unroll
            for (int i = 0; i < U; ++i) m = __builtin_fminf(m, t[i]);
        }
        const uint32_t s = wave_sort32(ordered_bits(m), lane);
        const uint32_t c = (uint32_t)__shfl((int)s, (ba.gather + NW - 1) / NW - 1, 64);
        if constexpr (NW == 1) {
            t1 = c;
        } else {
            if (lane == 0) wave_s[w] = c;
            __syncthreads();
            t1 = wave_s[0];
#pragma unroll
            for (int i = 1; i < NW; ++i) t1 = wave_s[i] > t1 ? wave_s[i] : t1;
        }
        const float t1f = t1 >= kInf ? 3.4028235e38f : from_ordered_bits(t1);   // (blocks without an entry, +inf, never pass)
        __syncthreads();
        auto take = [&](int64_t j) {
            const f32x4 v = fetch(j);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (v[e] <= t1f) {
                    const int pos = atomicAdd(&list_n, 1);
                    if (pos < kBlkList) list[pos] = ((uint64_t)ordered_bits(v[e]) << 32) | (uint32_t)(by_four ? j * 4 + e : j);
                }
            }
        };
        uint32_t hit = 0;   // groups of this thread that hold something
#pragma unroll
        for (int i = 0; i < G; ++i) hit |= (uint32_t)(gm[i] <= t1f) << i;
        while (hit) {
            const int i = __builtin_ctz(hit);
            hit &= hit - 1;
            take((int64_t)i * NT + tid);
        }
        for (int64_t j0 = (int64_t)G * NT + tid; j0 < ng; j0 += (int64_t)U * NT) {
            float t[U];
#pragma unroll
            for (int i = 0; i < U; ++i) t[i] = group_min(j0 + (int64_t)i * NT);
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (t[i] <= t1f) take(j0 + (int64_t)i * NT);
        }
    }
    __syncthreads();
    const int cnt = __builtin_amdgcn_readfirstlane(list_n);
    // (uniform) that many minima under T, which takes equal ones that the certificate could not tell apart
    // either; or none, which takes non-finite inputs; or, with T infinite, fewer than there are: the key of some
    // block's every entry overflowed, and those entries rank by their index
    if (cnt > kBlkList || cnt == 0 || (t1 >= kInf && cnt < ba.real_blocks)) {
        if (tid == 0) {
            a.flag_list2[atomicAdd(a.flag_count + 1, 1)] = q;
            if (a.stats) atomicAdd(a.stats + 2, 1ull);
        }
        return;
    }
    if (cnt <= 64) {
        if (w == 0) {
            const uint64_t x = wave_sort64(lane < cnt ? list[lane] : kSentinel, lane);
            list[lane] = x;
        }
        __syncthreads();
    } else {
        int n2 = 128;
        while (n2 < cnt) n2 <<= 1;
        for (int i = cnt + tid; i < n2; i += NT) list[i] = kSentinel;
        __syncthreads();
        bitonic_sort_lds(list, n2, tid, NT);
    }

    const float *qrow = a.queries + (int64_t)(a.sel ? a.sel[q] : q) * a.d;
    // slot 8 b + e: entry e of block b of the list
    auto entry_of = [&](int slot) { return block_first_entry((int)(uint32_t)list[slot >> 3]) + (slot & 3) + (slot >> 2 & 1) * 16; };
    if (NEXT && tid < RMAX && tid < cnt) {
        const uint32_t next = ba.bnext[(size_t)q * ba.nb + (uint32_t)list[tid]];
        others_s[tid] = block_others(from_ordered_bits((uint32_t)(list[tid] >> 32)), next);
        at_s[tid] = (uint8_t)(next & 7u);
    }
    bool ok = false;
    // first ba.first blocks, unconfirmed queries R, then all that were gathered
    // (where every block with an entry was gathered and they are hardly more, all at once: no certificate is needed
    // then.  19,804 points x 8, 128 centres, i.e. 16 blocks: 217 us a round with 8 first, 293 with 16 at once)
    int done = 0, nblk = cnt <= (t1 >= kInf ? ba.first + ba.first / 4 : ba.first) ? cnt : ba.first;
    nblk = nblk < RMAX ? nblk : RMAX;
    while (true) {
        // what is outside these blocks has a key above T, or at or above the next minimum (nothing is where T is infinite
        // and all blocks are taken)
        uint32_t excl = t1 >= kInf ? 0xffffffffu : t1;
        if (cnt > nblk) {
            const uint32_t nxt = (uint32_t)(list[nblk] >> 32);
            excl = nxt < excl ? nxt : excl;
        }
        const float exclf = excl >= kInf ? inf : from_ordered_bits(excl);
        // ---- 2. exact re-scoring: of blocks [done, nblk) the entry with the smallest key; of blocks whose other entries
        // may come before what is left out, all of them.  Packed (distance, index) by slot ----
        if constexpr (NEXT) {
            for (int i = done * 8 + tid; i < nblk * 8; i += NT) ent[i] = kSentinel;
            __syncthreads();
            if (w == 0) {   // a lane per block (RMAX of them at most); first the blocks of which one entry does
                const bool fresh = lane >= done && lane < nblk, open = lane < nblk && !(others_s[lane] >= exclf);   // (also no number)
                const uint64_t ones = __ballot(fresh && !open), wholes = __ballot(open), below = (1ull << lane) - 1ull;
                const int base = __builtin_popcountll(ones);
                if (fresh) {
                    const int slot = lane * 8 + at_s[lane];
                    sidx_s[lane] = entry_of(slot);
                    if (!open) work_s[__builtin_popcountll(ones & below)] = (uint16_t)slot;
                }
                if (open) {
                    const int at = base + 8 * __builtin_popcountll(wholes & below);
#pragma unroll
                    for (int e = 0; e < 8; ++e) work_s[at + e] = (uint16_t)(lane * 8 + e);
                    others_s[lane] = inf;   // done with
                }
                if (lane == 0) open_n = base + 8 * __builtin_popcountll(wholes);
            }
            __syncthreads();
            const int work = __builtin_amdgcn_readfirstlane(open_n);
            for (int c0 = 8 * w; c0 < work; c0 += 8 * NW) {
                auto slot = [&](int j) { return (int)work_s[c0 + j < work ? c0 + j : work - 1]; };
                auto entry = [&](int j) { return entry_of(slot(j)); };
                ListRows<decltype(entry)> rows{entry, {}};
#pragma unroll
                for (int j = 0; j < 8; ++j) rows.first[j] = __builtin_amdgcn_readfirstlane(entry(j));
                const uint64_t x = rescore_rows8(a, qrow, rows, lane);
                if ((lane & 7) == 0) ent[slot(lane >> 3)] = x;
            }
        } else {
            for (int b = done + w; b < nblk; b += NW) {
                uint64_t x = rescore_rows8(a, qrow, BlockRows{block_first_entry(__builtin_amdgcn_readfirstlane((int)(uint32_t)list[b]))}, lane);
                if ((lane & 7) == 0) ent[b * 8 + (lane >> 3)] = x;
                x = block_nearest(x);   // the certificate's sample
                if (lane == 0) {
                    // (a block that was taken holds a real entry; the marker only with non-finite inputs)
                    sidx_s[b] = (uint32_t)x < (uint32_t)a.n ? (int32_t)(uint32_t)x : 0;
                    sdist_s[b] = from_ordered_bits((uint32_t)(x >> 32));
                }
            }
        }
        if (tid == 0) {
            distinct_s = 0;
            near_n = 0;
        }
        __syncthreads();
        if constexpr (NEXT) {
            if (tid >= done && tid < nblk)   // the certificate's samples
                sdist_s[tid] = from_ordered_bits((uint32_t)(ent[tid * 8 + at_s[tid]] >> 32));
            __syncthreads();
        }

        // ---- 3. the k nearest ----
        // The k-th smallest of the blocks' nearest distances bounds the k-th neighbour: usually a few more
        // than k entries are left under it, and one wave sorts them.
        const int total = nblk * 8;
        uint64_t *res = ent2;
        int near = 1 << 30;
        if (a.k <= nblk) {   // uniform
            if (w == 0) {
                const uint64_t x = wave_sort64(
                    lane < nblk ? ((uint64_t)ordered_bits(sdist_s[lane]) << 32) | (uint32_t)sidx_s[lane] : kSentinel, lane);
                if (lane == a.k - 1) kth_s = x;
            }
            __syncthreads();
            const uint64_t kth = kth_s;
            for (int c = tid; c < total; c += NT) {
                const uint64_t x = ent[c];
                if (x <= kth) {
                    const int pos = atomicAdd(&near_n, 1);
                    if (pos < 64) ent2[pos] = x;
                }
            }
            __syncthreads();
            near = __builtin_amdgcn_readfirstlane(near_n);
        }
        if (near <= 64) {
            if (w == 0) ent2[lane] = wave_sort64(lane < near ? ent2[lane] : kSentinel, lane);
            __syncthreads();
        } else {   // all of them (a second round needs ent again: the sort works on a copy)
            int n2 = 64;
            while (n2 < total) n2 <<= 1;   // <= RMAX * 8
            for (int i = tid; i < n2; i += NT) ent2[i] = i < total ? ent[i] : kSentinel;
            __syncthreads();
            bitonic_sort_lds(ent2, n2, tid, NT);
        }
        if (tid < a.k) {
            const uint64_t x = res[tid];
            // with finite inputs the first k are real entries; a "no entry" marker maps to row 0
            const int32_t im = x == kSentinel ? 0 : (int32_t)(uint32_t)x;
            const float dm = from_ordered_bits((uint32_t)(x >> 32));
            a.out_nbr_idx[(int64_t)q * a.k + tid] = im;
            a.out_nbr_dist[(int64_t)q * a.k + tid] = dm;
            lab_s[tid] = a.labels[im];
            dsel_s[tid] = dm;
            best_s[tid] = x;
            if (tid == 0) nearest_s = im;
        }

        // ---- 4. the certificate ----
        ok = t1 >= kInf && nblk >= cnt;   // nothing is left out
        if (ok) {   // uniform
            __syncthreads();
            break;
        }
        if constexpr (!NEXT) {
            for (int b0 = done + w * 4; b0 < nblk; b0 += 4 * NW) {
                const float s1 = coarse_dot4(a, ba.mu, qrow, sidx_s, b0, nblk, lane);
                const int bj = b0 + (lane >> 4);
                if ((lane & 15) == 0 && bj < nblk) samp_s[bj] = (uint64_t)ordered_bits(__builtin_fmaf(-2.f, s1, ba.norm[sidx_s[bj]])) << 32;
            }
        }
        if (tid < nblk) {
            int twin = 0;
            for (int j = 0; j < tid; ++j) twin |= (sdist_s[j] == sdist_s[tid]);
            if (!twin) atomicAdd(&distinct_s, 1);
        }
        __syncthreads();
        ok = __builtin_amdgcn_readfirstlane(
                 (int)certificate(NEXT ? list : samp_s, sdist_s, nblk, dsel_s[a.k - 1], excl, distinct_s, tid, &verdict_s,
                                  NEXT ? 4.0 : 4.0 + 2.0 * ba.nk)) != 0;
        const int most = cnt < RMAX ? cnt : RMAX;
        if (ok || nblk >= most) break;   // uniform
        done = nblk;
        nblk = nblk < r && r < most ? r : most;
        __syncthreads();
    }
    if (__builtin_expect(!ok, 0)) {   // uniform (and out of the way of the instruction fetch)
        if (tid == 0) flagged_s = atomicAdd(a.flag_count, 1);
        __syncthreads();
        const int flagged = __builtin_amdgcn_readfirstlane(flagged_s);
        if (flagged < kMeetQueries) {
            if (tid == 0) a.flag_list[flagged] = q;   // (and counted in the statistics there)
        } else {
            // ---- 5. the 256 blocks with the smallest minima; the first nblk of them are done ----
            // T = the kTier1-th smallest of kBlkList group minima: at least that many blocks (or all) are <= T
            auto minimum = [&](int64_t blk) { return ((uint64_t)ordered_bits(bq[blk]) << 32) | (uint32_t)blk; };
            for (int g = tid; g < kBlkList; g += NT) {
                uint64_t m = kSentinel;
                for (int64_t blk = g; blk < ba.nb; blk += kBlkList) {
                    const uint64_t x = minimum(blk);
                    m = x < m ? x : m;
                }
                ent[g] = m;
            }
            if (tid == 0) list_n = 0;
            __syncthreads();
            bitonic_sort_lds(ent, kBlkList, tid, NT);
            const uint64_t t = ent[kTier1 - 1];
            const uint32_t tk = (uint32_t)(t >> 32);
            for (int64_t blk = tid; blk < ba.nb; blk += NT) {
                const uint64_t x = minimum(blk);
                if (x <= t && (uint32_t)(x >> 32) < kInf) {
                    const int pos = atomicAdd(&list_n, 1);
                    if (pos < kBlkList) list[pos] = x;
                }
            }
            __syncthreads();
            const int got = __builtin_amdgcn_readfirstlane(list_n);
            if (got <= kBlkList && (tk < kInf || got == ba.real_blocks)) {   // uniform; else the exact scan
                int n2 = 64;
                while (n2 < got) n2 <<= 1;
                for (int i = got + tid; i < n2; i += NT) list[i] = kSentinel;
                __syncthreads();
                bitonic_sort_lds(list, n2, tid, NT);
                const int all = got < kTier1 ? got : kTier1;
                // blocks between two merges, and between two certificates (NEXT: mostly one row each)
                constexpr int CH = NEXT ? 64 : 16, STEP = 64;
                static_assert(8 * CH + kMaxK <= RMAX * 16 && CH <= RMAX && CH <= NT, "ent, work_s");
                if constexpr (NEXT) {
                    // all eight where the others may come before what is left out of the `all` blocks (of the first nblk: all but
                    // the one that has been re-scored, where the others have not)
                    const uint32_t nxt = got > all ? (uint32_t)(list[all] >> 32) : 0xffffffffu, out = tk < nxt ? tk : nxt;
                    const float outf = out >= kInf ? inf : from_ordered_bits(out);
                    for (int i = tid; i < all; i += NT) {
                        const uint32_t next = ba.bnext[(size_t)q * ba.nb + (uint32_t)list[i]];
                        const float others = block_others(from_ordered_bits((uint32_t)(list[i] >> 32)), next);
                        const bool whole = !(others >= outf) && !(i < nblk && others_s[i] == inf);
                        at_s[i] = (uint8_t)((next & 7u) | (whole ? 8u : 0u));
                    }
                }
                for (int from = NEXT ? 0 : nblk, end = nblk;;) {
                    end = end + STEP < all ? end + STEP : all;
                    for (int c0 = from; c0 < end; c0 += CH) {
                        if (tid == 0) near_n = open_n = 0;
                        __syncthreads();
                        const uint64_t tau = best_s[a.k - 1];
                        if constexpr (NEXT) {
                            if (tid < CH && c0 + tid < end) {
                                const int b = c0 + tid, at = at_s[b] & 7;
                                const bool whole = at_s[b] & 8, fresh = b >= nblk;
                                int pos = atomicAdd(&open_n, (fresh ? 1 : 0) + (whole ? 7 : 0));
                                for (int e = 0; e < 8; ++e)
                                    if (e == at ? fresh : whole) work_s[pos++] = (uint16_t)(b * 8 + e);
                            }
                            __syncthreads();
                            const int work = __builtin_amdgcn_readfirstlane(open_n);   // <= 8 CH
                            for (int g0 = 8 * w; g0 < work; g0 += 8 * NW) {
                                auto slot = [&](int j) { return (int)work_s[g0 + j < work ? g0 + j : work - 1]; };
                                auto entry = [&](int j) { return entry_of(slot(j)); };
                                ListRows<decltype(entry)> rows{entry, {}};
#pragma unroll
                                for (int j = 0; j < 8; ++j) rows.first[j] = __builtin_amdgcn_readfirstlane(entry(j));
                                const uint64_t x = rescore_rows8(a, qrow, rows, lane);
                                if ((lane & 7) == 0 && g0 + (lane >> 3) < work) {
                                    if (x < tau) ent[atomicAdd(&near_n, 1)] = x;
                                    const int sl = slot(lane >> 3), b = sl >> 3;
                                    if ((sl & 7) == (at_s[b] & 7)) sdist_s[b] = from_ordered_bits((uint32_t)(x >> 32));
                                }
                            }
                        } else for (int b = c0 + w; b < c0 + CH && b < end; b += NW) {
                            const uint64_t x =
                                rescore_rows8(a, qrow, BlockRows{block_first_entry(__builtin_amdgcn_readfirstlane((int)(uint32_t)list[b]))}, lane);
                            if ((lane & 7) == 0 && x < tau) ent[atomicAdd(&near_n, 1)] = x;   // <= 8 CH
                            const uint64_t near = block_nearest(x);
                            if (lane == 0) {
                                sidx_s[b] = (uint32_t)near < (uint32_t)a.n ? (int32_t)(uint32_t)near : 0;
                                sdist_s[b] = from_ordered_bits((uint32_t)(near >> 32));
                            }
                        }
                        __syncthreads();
                        const int c = __builtin_amdgcn_readfirstlane(near_n);
                        if (c > 0) {   // uniform
                            int m2 = 2;
                            while (m2 < c + a.k) m2 <<= 1;   // <= RMAX * 16
                            for (int i = c + tid; i < m2; i += NT) ent[i] = i < c + a.k ? best_s[i - c] : kSentinel;
                            __syncthreads();
                            bitonic_sort_lds(ent, m2, tid, NT);
                            if (tid < a.k) best_s[tid] = ent[tid];
                        }
                        __syncthreads();
                    }
                    for (int b = from + w * 4; !NEXT && b < end; b += 4 * NW) {
                        const float dot = coarse_dot4(a, ba.mu, qrow, sidx_s, b, end, lane);
                        const int bj = b + (lane >> 4);
                        if ((lane & 15) == 0 && bj < end)
                            samp_s[bj] = (uint64_t)ordered_bits(__builtin_fmaf(-2.f, dot, ba.norm[sidx_s[bj]])) << 32;
                    }
                    if (tid == 0) distinct_s = 0;
                    __syncthreads();
                    if (tid < a.k) {
                        const uint64_t x = best_s[tid];
                        const int32_t im = x == kSentinel ? 0 : (int32_t)(uint32_t)x;
                        const float dm = from_ordered_bits((uint32_t)(x >> 32));
                        a.out_nbr_idx[(int64_t)q * a.k + tid] = im;
                        a.out_nbr_dist[(int64_t)q * a.k + tid] = dm;
                        lab_s[tid] = a.labels[im];
                        dsel_s[tid] = dm;
                        if (tid == 0) nearest_s = im;
                    }
                    for (int i = tid; i < end; i += NT) {
                        int twin = 0;
                        for (int j = 0; j < i; ++j) twin |= (sdist_s[j] == sdist_s[i]);
                        if (!twin) atomicAdd(&distinct_s, 1);
                    }
                    __syncthreads();
                    const uint32_t out = tk >= kInf ? 0xffffffffu : tk, nxt = got > end ? (uint32_t)(list[end] >> 32) : 0xffffffffu;
                    ok = __builtin_amdgcn_readfirstlane((int)certificate(NEXT ? list : samp_s, sdist_s, end, dsel_s[a.k - 1], nxt < out ? nxt : out,
                                                                         distinct_s, tid, &verdict_s, NEXT ? 4.0 : 4.0 + 2.0 * ba.nk)) != 0;
                    if (ok || end >= all) break;   // uniform
                    from = end;
                    __syncthreads();
                }
            }
            if (tid == 0) {
                if (!ok) a.flag_list2[atomicAdd(a.flag_count + 1, 1)] = q;
                if (a.stats) atomicAdd(a.stats + (ok ? 1 : 2), 1ull);
            }
        }
    } else if (tid == 0 && a.stats) {
        atomicAdd(a.stats + (nblk > r ? 1 : 0), 1ull);
    }
    decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
}

static int64_t real_blocks_of(int64_t n, int64_t n_pad)   // blocks that hold an entry
{
    int64_t real = (n_pad / kTileN - 1) * (kTileN / 8);
    for (int blk = 0; blk < kTileN / 8; ++blk) real += n_pad - kTileN + block_first_entry(blk) < n;
    return real;
}

hipError_t launch_block_finish(const FinishArgs &a, const BlockMinima &m, hipStream_t s)
{
    const int64_t n_pad = m.n_pad;
    if (!m.bkey || a.r < 1 || a.r > kMaxRescore || a.k > kMaxK || a.k > a.r || a.b < 1 || !a.flag_count || !a.flag_list || !a.flag_list2 || n_pad % kTileN != 0)
        return hipErrorInvalidValue;
    // two blocks more than neighbours confirm most queries (4,096 x 50,000 x 512, k = 10, whole blocks: 112 us with 12 at
    // first, 118 with 11, 119 with 14, 129 with 16); the certificate wants eight samples at least
    int first = a.k + 2 > kCertMinSamples ? a.k + 2 : kCertMinSamples;
    first = first < a.r ? first : a.r;
    const int gather = 2 * a.r < kMaxRescore ? 2 * a.r : kMaxRescore;
    BlockFinishArgs ba{a, m.bkey, m.bnext, m.norm, m.mu, n_pad / 8, real_blocks_of(a.n, n_pad), (int)(a.d_pad / kKB), first, gather};
    // Two waves per query where the batch fills the chip with them, four where it does not (50,000 x 512: 1,500
    // queries 54 against 59 us, 600 queries 42 against 34 us; one wave per query is slower than two at both).
    if (a.b >= 1024 && m.bnext)
        hipLaunchKernelGGL((block_finish_kernel<128, true>), dim3((unsigned)a.b), dim3(128), 0, s, ba);
    else if (a.b >= 1024)
        hipLaunchKernelGGL((block_finish_kernel<128, false>), dim3((unsigned)a.b), dim3(128), 0, s, ba);
    else if (m.bnext)
        hipLaunchKernelGGL((block_finish_kernel<256, true>), dim3((unsigned)a.b), dim3(256), 0, s, ba);
    else
        hipLaunchKernelGGL((block_finish_kernel<256, false>), dim3((unsigned)a.b), dim3(256), 0, s, ba);
    return hipGetLastError();
}

hipError_t launch_finish(const FinishArgs &a, hipStream_t s)
{
    const int total = a.alloc_splits * a.r;   // (candidate lists with a count are keys_finish_kernel's)
    if (a.part_count || total > kMaxMergeEntries || a.r > kMaxRescore || a.k > kMaxK || a.k > a.r) return hipErrorInvalidValue;
    if (!a.flag_count || !a.flag_list || !a.flag_list2) return hipErrorInvalidValue;
    // (the second step takes sixteen candidates at most: a loop there costs the whole kernel registers)
    const int first = first_width(a, true);
    FinishKernelArgs fa{a, 2, first > a.r - 16 ? first : a.r - 16};
    while (fa.sort_cap < total) fa.sort_cap <<= 1;
    const size_t lds = (size_t)fa.sort_cap * sizeof(uint64_t);
    // a block per query: with few queries and long activations use 1024-thread blocks
    if (wide_order(a.b, a.d))
        hipLaunchKernelGGL((finish_kernel<1024>), dim3((unsigned)a.b), dim3(1024), lds, s, fa);
    else
        hipLaunchKernelGGL((finish_kernel<256>), dim3((unsigned)a.b), dim3(256), lds, s, fa);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Follow-up of a look-up, one launch: the queries whose result the certificate did not confirm.
// Nothing is flagged on the paper's kind of data, and then the kernel reads two counters and returns;
// an empty launch costs 4.6 us and the gap before it, so the two rounds share one (256 x 2,000 x 512: whole
// look-up 26.0 -> 24.4 us).
//
// Round 1, the wider re-scoring (list 0): up to kTier1 of the candidates gathered by the distance pass, or of
// the blocks with the smallest minima, are re-scored and the certificate is taken again.  Workgroups take items off a queue: a query, or, with
// few flagged queries, a sixteenth of a query's candidates; the last of its sixteen to finish (a ticket
// per query) decides.  (One request of a 65,536-value layer, 32 MB of rows, kept a single workgroup busy
// for 630 us; shared it takes 70.  20 queries
// of 512 values: 63 -> 48 us.)  What is still unconfirmed goes on list 1.
// A workgroup that finds the queue empty waits until every item taken off it is done: those are all held
// by running workgroups, which wait for nothing while they hold one, so the wait ends whatever part of
// the grid is resident.
//
// Round 2, the exact scan (list 1; Sec. 3: the look-up returns THE k nearest neighbours):
// brute-force fp32 distances sum (q_i - c_i)^2 to every stored entry, the same arithmetic as the
// re-scoring above, no bf16 anywhere.  The grid shares the flagged queries: with nf of them, each is cut
// into S = grid / nf ranges of at least 16 entries (at least one range, at most max_splits); a workgroup
// scans its range 256 entries at a time and keeps the k nearest by (distance, index); the last workgroup
// of a query to finish (a ticket per query) merges the S lists and writes the neighbours, the label and
// the hit decision over that query's outputs.
// ---------------------------------------------------------------------------------------
struct ScanArgs {
    FinishArgs a;
    int32_t *tickets;    // [b], zero on entry; left zero
    uint64_t *part_x;    // [items, k] the k nearest of each (query, range), packed (ordered distance, index)
    int max_splits;
    int64_t part_bytes;  // size of part_x
    // block-minima route (else null / unused): the smallest coarse key of every block, as in BlockFinishArgs
    const float *bkey, *norm, *mu;
    int64_t nb, real_blocks;
    int nk;
    uint64_t *meet;      // [kMeetQueries, kWiderParts, kMeetEntries] what the workgroups that share a query pass on
};
constexpr int kMeetSamples = kTier1 / kWiderParts, kMeetEntries = kMaxK + kMeetSamples;
constexpr int kWiderList = 1024;   // block minima gathered for the wider re-scoring at most

__global__ __launch_bounds__(256) void follow_up_kernel(ScanArgs sa)
{
    const FinishArgs &a = sa.a;
    extern __shared__ uint64_t ent[];   // >= 512 entries, >= max_splits * k, >= the gathered candidates of a query
    __shared__ float red[4][8];
    __shared__ float dist_s[256];
    __shared__ int32_t idx_s[256];
    __shared__ uint64_t best_s[kMaxK];
    __shared__ int32_t lab_s[kMaxK];
    __shared__ int32_t cnt_s[kMaxK];
    __shared__ float dsel_s[kMaxK];
    __shared__ double conf_s[kMaxK];
    __shared__ int32_t nearest_s;
    __shared__ int surv_s, last_s, job_s, real_s, distinct_s, verdict_s;
    __shared__ uint32_t excl_s;

    const int flagged = a.flag_count[0];
    int nf = a.flag_count[1];
    if (flagged <= 0 && nf <= 0) return;   // the usual case
    // (of block minima only the first kMeetQueries flagged queries are left to this kernel)
    const int n_wider = sa.bkey && flagged > kMeetQueries ? kMeetQueries : flagged;
    const int tid = threadIdx.x;
    const int grid = (int)gridDim.x, k = a.k;

    // ---- round 1: wider re-scoring ----
    if (n_wider > 0) {   // uniform
        const int nq = a.count ? *a.count : a.b;
        // few flagged queries: kWiderParts workgroups share each, the distances meet in round 2's scratch
        const bool split = n_wider * kWiderParts <= grid &&
                           (sa.bkey || (int64_t)n_wider * kTier1 * 4 <= sa.part_bytes);
        const int items = split ? n_wider * kWiderParts : n_wider;
        bool held = false;   // an item taken off the queue is finished, but not yet counted
        while (true) {
            // (thread 0 counts the last item and takes the next in one place, with barriers on both sides: a
            // branch of thread 0 at the loop's end and another at its top would be joined by the compiler into
            // a path on which the other threads run ahead to the next barrier)
            if (tid == 0) {
                if (held) atomicAdd(a.flag_count + 3, 1);
                job_s = atomicAdd(a.flag_count + 2, 1);
            }
            __syncthreads();
            const int job = __builtin_amdgcn_readfirstlane(job_s);
            if (job >= items) break;   // uniform
            held = true;
            const int j = split ? job / kWiderParts : job;
            const int q = __builtin_amdgcn_readfirstlane(a.flag_list[j]);
            const float *qrow = a.queries + (int64_t)(a.sel ? a.sel[q] : q) * a.d;
            bool mine = true, ok = false;   // mine: this workgroup decides the query
            if (sa.bkey) {   // uniform
                // Selection: the 1,024 groups j mod 1,024 of the block minima; T = the kTier1-th smallest group
                // minimum, so that at least kTier1 blocks (or all) have a minimum <= T.  Blocks of +inf hold padding, or
                // entries whose key overflowed, and are not taken.
                const float *bq = sa.bkey + (size_t)q * sa.nb;
                constexpr uint32_t kInf = 0xff800000u;
                auto minimum = [&](int64_t blk) { return ((uint64_t)ordered_bits(bq[blk]) << 32) | (uint32_t)blk; };
                for (int g = tid; g < 1024; g += 256) {
                    uint64_t m = kSentinel;
                    for (int64_t blk = g; blk < sa.nb; blk += 1024) {
                        const uint64_t x = minimum(blk);
                        m = x < m ? x : m;
                    }
                    ent[g] = m;
                }
                if (tid == 0) surv_s = 0;
                __syncthreads();
                bitonic_sort_lds(ent, 1024, tid, 256);
                const uint64_t t = ent[kTier1 - 1];
                const uint32_t tk = (uint32_t)(t >> 32);
                uint64_t *blocks = ent + 1024;         // [kWiderList] what is gathered, in order
                uint64_t *samples = ent + 1024 + kWiderList;   // [kTier1] coarse keys (upper halves) of the blocks' nearest entries
                for (int64_t blk = tid; blk < sa.nb; blk += 256) {
                    const uint64_t x = minimum(blk);
                    if (x <= t && (uint32_t)(x >> 32) < kInf) {
                        const int pos = atomicAdd(&surv_s, 1);
                        if (pos < kWiderList) blocks[pos] = x;
                    }
                }
                __syncthreads();
                const int cnt = __builtin_amdgcn_readfirstlane(surv_s);
                // more than fit, or entries whose key overflowed are left out: the exact scan
                const bool sound = cnt <= kWiderList && (tk < kInf || cnt == sa.real_blocks);
                const int nblk = !sound ? 0 : (cnt < kTier1 ? cnt : kTier1);
                if (sound) {   // uniform
                    int n2 = 64;
                    while (n2 < cnt) n2 <<= 1;
                    for (int i = cnt + tid; i < n2; i += 256) blocks[i] = kSentinel;
                    __syncthreads();
                    bitonic_sort_lds(blocks, n2, tid, 256);
                }
                // exact re-scoring, sixteen blocks at a time: their nearest entries as samples, the k nearest of all
                const int w = tid >> 6, lane = tid & 63, part = split ? job % kWiderParts : 0;
                const int p0 = part * kMeetSamples, p1 = split && p0 + kMeetSamples < nblk ? p0 + kMeetSamples : nblk;
                if (tid < kMaxK) best_s[tid] = kSentinel;
                for (int b0 = p0; b0 < p1; b0 += kMeetSamples) {
                    if (tid == 0) surv_s = 0;
                    __syncthreads();
                    const int b1 = b0 + kMeetSamples < p1 ? b0 + kMeetSamples : p1;
                    const uint64_t tau = best_s[k - 1];
                    for (int b = b0 + w; b < b1; b += 4) {
                        const uint64_t x =
                            rescore_rows8(a, qrow, BlockRows{block_first_entry(__builtin_amdgcn_readfirstlane((int)(uint32_t)blocks[b]))}, lane);
                        if ((lane & 7) == 0 && x < tau) ent[atomicAdd(&surv_s, 1)] = x;   // <= 128
                        const uint64_t near = block_nearest(x);
                        if (lane == 0) {
                            idx_s[b] = (uint32_t)near < (uint32_t)a.n ? (int32_t)(uint32_t)near : 0;
                            dist_s[b] = from_ordered_bits((uint32_t)(near >> 32));
                        }
                    }
                    __syncthreads();
                    const int c = __builtin_amdgcn_readfirstlane(surv_s);
                    if (c > 0) {   // uniform
                        int n2 = 2;
                        while (n2 < c + k) n2 <<= 1;   // <= 256
                        for (int i = c + tid; i < n2; i += 256) ent[i] = i < c + k ? best_s[i - c] : kSentinel;
                        __syncthreads();
                        bitonic_sort_lds(ent, n2, tid, 256);
                        if (tid < k) best_s[tid] = ent[tid];
                    }
                    __syncthreads();
                }
                for (int b0 = p0 + w * 4; b0 < p1; b0 += 16) {
                    const float dot = coarse_dot4(a, sa.mu, qrow, idx_s, b0, p1, lane);
                    const int bj = b0 + (lane >> 4);
                    if ((lane & 15) == 0 && bj < p1)
                        samples[bj] = (uint64_t)ordered_bits(__builtin_fmaf(-2.f, dot, sa.norm[idx_s[bj]])) << 32;
                }
                __syncthreads();
                if (split) {
                    uint64_t *meet = sa.meet + (size_t)j * kWiderParts * kMeetEntries, *own = meet + part * kMeetEntries;
                    if (tid < k) __hip_atomic_store(own + tid, best_s[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (p0 + tid < p1 && tid < kMeetSamples)
                        __hip_atomic_store(own + kMaxK + tid, samples[p0 + tid] | __float_as_uint(dist_s[p0 + tid]), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    if (tid == 0) {
                        last_s = (atomicAdd(&sa.tickets[j], 1) == kWiderParts - 1);
                        if (last_s) atomicExch(&sa.tickets[j], 0);   // round 2 finds it zero
                    }
                    __syncthreads();
                    mine = __builtin_amdgcn_readfirstlane(last_s) != 0;
                    if (mine) {
                        for (int i = tid; i < 1024; i += 256)
                            ent[i] = i < kWiderParts * k ? __hip_atomic_load(meet + i / k * kMeetEntries + i % k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                                         : kSentinel;
                        if (tid < nblk) {
                            const uint64_t sv = __hip_atomic_load(meet + tid / kMeetSamples * kMeetEntries + kMaxK + tid % kMeetSamples,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                            samples[tid] = sv & 0xffffffff00000000ull;
                            dist_s[tid] = __uint_as_float((uint32_t)sv);
                        }
                        __syncthreads();
                        bitonic_sort_lds(ent, 1024, tid, 256);
                        if (tid < k) best_s[tid] = ent[tid];
                        __syncthreads();
                    }
                }
                if (mine) {   // uniform
                    if (tid == 0) distinct_s = 0;
                    __syncthreads();
                    if (tid < k) {
                        const uint64_t x = best_s[tid];   // (a marker only where nothing sound was selected: the exact scan follows)
                        const int32_t im = x == kSentinel ? 0 : (int32_t)(uint32_t)x;
                        const float dm = from_ordered_bits((uint32_t)(x >> 32));
                        a.out_nbr_idx[(int64_t)q * k + tid] = im;
                        a.out_nbr_dist[(int64_t)q * k + tid] = dm;
                        lab_s[tid] = a.labels[im];
                        dsel_s[tid] = dm;
                        if (tid == 0) nearest_s = im;
                    }
                    if (tid < nblk) {
                        int twin = 0;
                        for (int i = 0; i < tid; ++i) twin |= (dist_s[i] == dist_s[tid]);
                        if (!twin) atomicAdd(&distinct_s, 1);
                    }
                    __syncthreads();
                    const uint32_t out = tk >= kInf ? 0xffffffffu : tk;
                    const uint32_t nxt = cnt > nblk && sound ? (uint32_t)(blocks[nblk] >> 32) : 0xffffffffu;
                    ok = sound && __builtin_amdgcn_readfirstlane((int)certificate(samples, dist_s, nblk, dsel_s[k - 1], nxt < out ? nxt : out,
                                                                                  distinct_s, tid, &verdict_s, 4.0 + 2.0 * sa.nk)) != 0;
                }
            } else {
                const int total = gather_entries(a, q, nq, ent, &real_s, &excl_s, tid, 256);
                int sort_n = 2;
                while (sort_n < total) sort_n <<= 1;
                bitonic_sort_lds(ent, sort_n, tid, 256);
                const int real = __builtin_amdgcn_readfirstlane(real_s);
                const int most = real < kTier1 ? real : kTier1;   // (real entries sort in front of the markers)
                const bool whole_block = a.d >= 4096 && a.d % 8 == 0;
                // a candidate list (keys-out routes) holds every entry up to its largest pair
                const uint32_t excl0 = a.part_count ? (real >= a.n || real < 1 ? 0xffffffffu : (uint32_t)(ent[real - 1] >> 32)) : excl_s;
                if (tid < most) idx_s[tid] = (int32_t)(uint32_t)ent[tid];   // < n: counted as real
                __syncthreads();
                auto rescore = [&](int m0, int m) {   // candidates [m0, m)
                    if (whole_block) {
                        for (int c0 = m0; c0 < m; c0 += 16)
                            rescore_block_any<16>(a, qrow, idx_s + c0, dist_s + c0, red, m - c0 < 16 ? m - c0 : 16, tid);
                    } else {
                        // (sixteen rows in flight per wave where there are enough: 4,538 x 29,747 fp32, 47 queries 901 us, 1,474 with four)
                        if (m - m0 > 32) rescore_wave<16>(a, qrow, idx_s + m0, dist_s + m0, m - m0, tid >> 6, tid & 63);
                        else rescore_wave<4>(a, qrow, idx_s + m0, dist_s + m0, m - m0, tid >> 6, tid & 63);
                        __syncthreads();
                    }
                };
                auto confirm = [&](int m) {
                    if (tid == 0) distinct_s = 0;
                    __syncthreads();
                    rank_and_emit(a, q, m, tid, 256, dist_s, idx_s, lab_s, dsel_s, &nearest_s, &distinct_s);
                    __syncthreads();
                    uint32_t excl = excl0;
                    if (real > m) {
                        const uint32_t nxt = (uint32_t)(ent[m] >> 32);
                        excl = nxt < excl ? nxt : excl;
                    }
                    return __builtin_amdgcn_readfirstlane(
                               (int)certificate(ent, dist_s, m, dsel_s[k - 1], excl, distinct_s, tid, &verdict_s)) != 0;
                };
                if (split) {
                    constexpr int per = kTier1 / kWiderParts;
                    float *meet = reinterpret_cast<float *>(sa.part_x) + (size_t)j * kTier1;
                    const int m0 = (job % kWiderParts) * per, m = m0 + per < most ? m0 + per : most;
                    if (m0 < m) rescore(m0, m);
                    // device-coherent stores, complete before the ticket is taken, and device-coherent loads: no fence,
                    // which would write back the whole L2 (a fence per wave took 100 us in place of 45 on 20 queries)
                    if (tid >= m0 && tid < m) __hip_atomic_store(meet + tid, dist_s[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    __syncthreads();
                    if (tid == 0) {
                        last_s = (atomicAdd(&sa.tickets[j], 1) == kWiderParts - 1);
                        if (last_s) atomicExch(&sa.tickets[j], 0);   // round 2 finds it zero
                    }
                    __syncthreads();
                    mine = __builtin_amdgcn_readfirstlane(last_s) != 0;
                    if (mine) {
                        if (tid < most) dist_s[tid] = __hip_atomic_load(meet + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        ok = confirm(most);
                    }
                } else {
                    // many flagged queries: a workgroup each; of long rows twice as many at a time, until the
                    // certificate, whose bound grows with the first key left out, confirms the result
                    for (int m0 = 0, m = whole_block ? 64 : most; !ok && m0 < most; m0 = m, m *= 2) {
                        m = m < most ? m : most;
                        rescore(m0, m);
                        ok = confirm(m);
                    }
                }
            }
            if (mine) {
                if (tid == 0) {
                    if (!ok)
                        __hip_atomic_store(a.flag_list2 + atomicAdd(a.flag_count + 1, 1), q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (a.stats) atomicAdd(a.stats + (ok ? 1 : 2), 1ull);
                }
                decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
                // round 2 overwrites the outputs of an unconfirmed query, perhaps from another XCD: these
                // stores leave this one's L2 before the query counts as done
                if (!ok) __threadfence();
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        __syncthreads();
        if (tid == 0)
            while (__hip_atomic_load(a.flag_count + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < items) __builtin_amdgcn_s_sleep(16);
        __syncthreads();
        nf = __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.flag_count + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (nf <= 0) return;   // uniform
    }

    // ---- round 2: exact scan ----
    int S = grid / nf;
    const int by_size = (a.n + 15) / 16;   // a range holds at least 16 entries
    S = S > sa.max_splits ? sa.max_splits : S;
    S = S > by_size ? by_size : S;
    S = S < 1 ? 1 : S;
    const int64_t items = (int64_t)nf * S;
    for (int64_t item = blockIdx.x; item < items; item += grid) {
        const int j = (int)(item / S), sp = (int)(item - (int64_t)j * S);
        const int q = __builtin_amdgcn_readfirstlane(__hip_atomic_load(a.flag_list2 + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        const float *qrow = a.queries + (int64_t)(a.sel ? a.sel[q] : q) * a.d;
        const int row0 = (int)((int64_t)a.n * sp / S), row1 = (int)((int64_t)a.n * (sp + 1) / S);
        if (tid < kMaxK) best_s[tid] = kSentinel;
        __syncthreads();
        for (int base = row0; base < row1; base += 256) {
            const int m = row1 - base < 256 ? row1 - base : 256;
            if (tid < m) idx_s[tid] = base + tid;
            if (tid == 0) surv_s = 0;
            __syncthreads();
            if (a.d >= 4096 && a.d % 8 == 0) {
                for (int c0 = 0; c0 < m; c0 += 32)
                    rescore_block_any<32>(a, qrow, idx_s + c0, dist_s + c0, red, m - c0 < 32 ? m - c0 : 32, tid);
            } else
                rescore_wave<16>(a, qrow, idx_s, dist_s, m, tid >> 6, tid & 63);
            __syncthreads();
            // entries that beat the k-th best so far, then the k best of those and the list
            const uint64_t tau = best_s[k - 1];
            if (tid < m) {
                const uint64_t x = ((uint64_t)ordered_bits(dist_s[tid]) << 32) | (uint32_t)(base + tid);
                if (x < tau) ent[atomicAdd(&surv_s, 1)] = x;
            }
            __syncthreads();
            const int c = surv_s;
            if (c > 0) {   // uniform
                int n2 = 2;
                while (n2 < c + k) n2 <<= 1;   // <= 512
                for (int i = c + tid; i < n2; i += 256) ent[i] = i < c + k ? best_s[i - c] : kSentinel;
                __syncthreads();
                bitonic_sort_lds(ent, n2, tid, 256);
                if (tid < k) best_s[tid] = ent[tid];
                __syncthreads();
            }
        }
        if (tid < k) sa.part_x[(size_t)item * k + tid] = best_s[tid];
        __syncthreads();
        if (tid == 0) {
            __threadfence();   // the list is visible to the whole device before the ticket is taken
            last_s = (atomicAdd(&sa.tickets[j], 1) == S - 1);
            __threadfence();
        }
        __syncthreads();
        if (last_s) {   // uniform: this workgroup finished the query's last range
            // The lists are sorted.  The k-th smallest of their heads (of S >= k lists) bounds the k-th entry:
            // k lists have a head at or under it, so at most k * k entries are, usually a few more than k.
            // (A sort of all S * k took 150 us of a scan of 50,000 x 1,024; up to 1,024 entries it is the shorter way:
            // 68,906 x 2, k = 1, 86 us for the scan with the heads ranked first, 48 without.)
            const int total = S * k;
            const uint64_t *src = sa.part_x + (size_t)j * S * k;
            uint64_t bound = kSentinel;
            if (S > k && total > 1024) {   // uniform
                int h2 = 2;
                while (h2 < S) h2 <<= 1;   // <= kScanMaxSplits
                for (int i = tid; i < h2; i += 256)
                    ent[i] = i < S ? __hip_atomic_load(src + (size_t)i * k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kSentinel;
                __syncthreads();
                bitonic_sort_lds(ent, h2, tid, 256);
                bound = ent[k - 1];
                __syncthreads();
            }
            if (tid == 0) surv_s = 0;
            __syncthreads();
            for (int i = tid; i < total; i += 256) {
                const uint64_t x = __hip_atomic_load(src + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (x <= bound) ent[atomicAdd(&surv_s, 1)] = x;
            }
            __syncthreads();
            const int got = __builtin_amdgcn_readfirstlane(surv_s);
            int n2 = 2;
            while (n2 < got || n2 < k) n2 <<= 1;   // got <= total <= the allocation
            for (int i = got + tid; i < n2; i += 256) ent[i] = kSentinel;
            __syncthreads();
            bitonic_sort_lds(ent, n2, tid, 256);
            if (tid < k) {
                const uint64_t x = ent[tid];
                const int32_t im = (uint32_t)x < (uint32_t)a.n ? (int32_t)(uint32_t)x : 0;   // (non-finite inputs only)
                const float dm = from_ordered_bits((uint32_t)(x >> 32));
                a.out_nbr_idx[(int64_t)q * k + tid] = im;
                a.out_nbr_dist[(int64_t)q * k + tid] = dm;
                lab_s[tid] = a.labels[im];
                dsel_s[tid] = dm;
                if (tid == 0) {
                    nearest_s = im;
                    sa.tickets[j] = 0;
                }
            }
            __syncthreads();
            decide_and_write(a, q, tid, lab_s, dsel_s, cnt_s, conf_s, nearest_s);
        }
        __syncthreads();
    }
}

static int scan_max_splits(int k) { return kMaxMergeEntries / k < kScanMaxSplits ? kMaxMergeEntries / k : kScanMaxSplits; }
// (an empty launch costs the same 4 us whatever its grid: no smaller grid for small batches, whose
// flagged queries then get all the workgroups)
static int scan_grid(int num_cus, int64_t) { return 2 * num_cus; }

size_t scan_scratch_entries(int64_t b, int k, int num_cus)
{
    // items = flagged queries x ranges <= max(b, grid)
    const int64_t items = b > scan_grid(num_cus, b) ? b : scan_grid(num_cus, b);
    return (size_t)items * (size_t)k;
}

size_t follow_up_meet_entries() { return (size_t)kMeetQueries * kWiderParts * kMeetEntries; }

hipError_t launch_follow_up(const FinishArgs &a, int32_t *tickets, uint64_t *part_x, int num_cus, const BlockMinima *blocks, hipStream_t s)
{
    if (!a.flag_count || !a.flag_list || !a.flag_list2 || !tickets || !part_x || a.k < 1 || a.k > kMaxK) return hipErrorInvalidValue;
    const int total = a.part_count ? a.part_stride : a.alloc_splits * a.r;   // (0: block minima, or nothing goes on list 0)
    if (total > kMaxMergeEntries) return hipErrorInvalidValue;
    const int grid = scan_grid(num_cus, a.b);
    ScanArgs sa{a, tickets, part_x, scan_max_splits(a.k) < grid ? scan_max_splits(a.k) : grid,
                (int64_t)(scan_scratch_entries(a.b, a.k, num_cus) * 8)};
    int cap = 512;
    if (blocks) {
        if (!blocks->bkey || !blocks->norm || !blocks->meet || total != 0) return hipErrorInvalidValue;
        sa.bkey = blocks->bkey;
        sa.norm = blocks->norm;
        sa.mu = blocks->mu;
        sa.nb = blocks->n_pad / 8;
        sa.real_blocks = real_blocks_of(a.n, blocks->n_pad);
        sa.nk = (int)(a.d_pad / kKB);
        sa.meet = blocks->meet;
        static_assert(1024 + kWiderList + kTier1 <= 4096, "group minima, blocks, samples");
        cap = 4096;
    }
    while (cap < sa.max_splits * a.k || cap < total) cap <<= 1;   // (a power of two: the sorts pad to one)
    hipLaunchKernelGGL(follow_up_kernel, dim3((unsigned)grid), dim3(256), (size_t)cap * sizeof(uint64_t), s, sa);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Miss compaction (Sec. 5, "Freeze Inference on GPUs": the batch is rebuilt without the
// frozen items).  Stable: misses keep their order.  One block; ballot-based scan.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void compact_kernel(const uint8_t *hit, const int32_t *sel_in, const int32_t *count_in,
                                                       int count_max, int32_t *sel_out, int32_t *count_out,
                                                       int64_t *hits_out)
{
    __shared__ int wave_tot[16];
    __shared__ int base_s;
    const int cnt = count_in ? *count_in : count_max;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) base_s = 0;
    __syncthreads();
    for (int start = 0; start < cnt; start += 1024) {
        const int j = start + tid;
        const bool miss = (j < cnt) && (hit[j] == 0);
        const uint64_t bal = __ballot(miss);
        const int before = __builtin_popcountll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wave_tot[w] = __builtin_popcountll(bal);
        __syncthreads();
        int off = base_s;
        for (int i = 0; i < w; ++i) off += wave_tot[i];
        if (miss) sel_out[off + before] = sel_in ? sel_in[j] : j;
        __syncthreads();
        if (tid == 0) {
            int t = 0;
            for (int i = 0; i < 16; ++i) t += wave_tot[i];
            base_s += t;
        }
        __syncthreads();
    }
    if (tid == 0) {
        *count_out = base_s;
        if (hits_out) *hits_out = (int64_t)cnt - (int64_t)base_s;
    }
}

hipError_t launch_compact(const uint8_t *hit, const int32_t *sel_in, const int32_t *count_in, int64_t count_max,
                          int32_t *sel_out, int32_t *count_out, int64_t *hits_out, hipStream_t s)
{
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, s, hit, sel_in, count_in, (int)count_max, sel_out,
                       count_out, hits_out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Cascade bookkeeping (Pseudocode 1, FreezeInference): start with "no layer hit", then
// after each layer record (label, layer position) for the requests that hit there.
// ---------------------------------------------------------------------------------------
__global__ void cascade_init_kernel(int32_t *out_labels, int32_t *out_exit, int64_t b)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < b) {
        out_labels[i] = -1;
        out_exit[i] = -1;
    }
}

hipError_t launch_cascade_init(int32_t *out_labels, int32_t *out_exit, int64_t b, hipStream_t s)
{
    hipLaunchKernelGGL(cascade_init_kernel, dim3((unsigned)((b + 255) / 256)), dim3(256), 0, s, out_labels, out_exit, b);
    return hipGetLastError();
}

__global__ void cascade_scatter_kernel(const int32_t *labels, const uint8_t *hit, const int32_t *sel, const int32_t *count,
                                       int b, int layer_pos, int32_t *out_labels, int32_t *out_exit)
{
    const int nq = count ? *count : b;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nq && hit[j]) {
        const int orig = sel ? sel[j] : j;
        out_labels[orig] = labels[j];
        out_exit[orig] = layer_pos;
    }
}

hipError_t launch_cascade_scatter(const int32_t *labels, const uint8_t *hit, const int32_t *sel,
                                  const int32_t *count, int64_t b, int layer_pos, int32_t *out_labels,
                                  int32_t *out_exit, hipStream_t s)
{
    hipLaunchKernelGGL(cascade_scatter_kernel, dim3((unsigned)((b + 255) / 256)), dim3(256), 0, s, labels, hit, sel,
                       count, (int)b, layer_pos, out_labels, out_exit);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Batch reconstruction of a tensor (Sec. 5, "Freeze Inference on GPUs"): the rows of the missed
// requests, in miss-list order, so that the next layer of the model runs on a dense smaller
// batch.  One block per output row; nothing is done past the device-side count.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gather_rows_kernel(const float *x, int64_t d, const int32_t *sel, const int32_t *count,
                                                          int64_t max_count, float *out)
{
    const int64_t nq = count ? *count : max_count;
    const int64_t j = blockIdx.x;
    if (j >= nq) return;
    const float *src = x + (int64_t)sel[j] * d;
    float *dst = out + j * d;
    if ((d % 4) == 0 && (reinterpret_cast<uintptr_t>(x) % 16) == 0 && (reinterpret_cast<uintptr_t>(out) % 16) == 0) {
        for (int64_t i = threadIdx.x; i < d / 4; i += 256)
            reinterpret_cast<f32x4 *>(dst)[i] = reinterpret_cast<const f32x4 *>(src)[i];
    } else {
        for (int64_t i = threadIdx.x; i < d; i += 256) dst[i] = src[i];
    }
}

hipError_t launch_gather_rows(const float *x, int64_t d, const int32_t *sel, const int32_t *count, int64_t max_count,
                              float *out, hipStream_t s)
{
    if (max_count <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)max_count), dim3(256), 0, s, x, d, sel, count, max_count, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------
// Per-layer threshold (Pseudocode 1, ComputeThresholds): the largest confidence among the
// validation items whose look-up disagrees with the model's label; 0 when none disagrees.
// Confidences are >= 0 (or +inf), so their fp32 bit patterns order like unsigned integers.
// ---------------------------------------------------------------------------------------
__global__ void threshold_init_kernel(float *thr, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) thr[i] = 0.f;
}

__global__ void threshold_max_kernel(const int32_t *pred, const float *conf, const int32_t *model_labels, int64_t b,
                                     float *thr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t v = 0;
    if (i < b && pred[i] != model_labels[i]) v = __float_as_uint(conf[i]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)v, off, 64);
        v = o > v ? o : v;
    }
    if ((threadIdx.x & 63) == 0 && v != 0) atomicMax(reinterpret_cast<unsigned int *>(thr), v);
}

hipError_t launch_threshold_init(float *thr, int n, hipStream_t s)
{
    hipLaunchKernelGGL(threshold_init_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, thr, n);
    return hipGetLastError();
}

hipError_t launch_threshold_max(const int32_t *pred, const float *conf, const int32_t *model_labels, int64_t b,
                                float *thr, hipStream_t s)
{
    if (b <= 0) return hipSuccess;
    hipLaunchKernelGGL(threshold_max_kernel, dim3((unsigned)((b + 255) / 256)), dim3(256), 0, s, pred, conf,
                       model_labels, b, thr);
    return hipGetLastError();
}

}  // namespace fz
