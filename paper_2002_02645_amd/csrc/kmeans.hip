// k-means cache (paper Sec. 4, "k-means"): the intermediate points of a layer are clustered
// and each cluster is represented by its centre; a cache item is the centre, the majority
// label of the cluster and the fraction of the cluster that carries it.
//
// The assignment step of Lloyd's iterations is a product of the points with split centres (rows_gemm.hip) from 256
// points and up to 512 centres; else, and in a workspace without room for its sums, the batched look-up (every point
// against the centres, k = 1).  Both are driven from the API file; this file holds what is left: the update of the
// centres, the majority label and fraction of every cluster, and a read-out.  gfx950 only.
#include "freeze_internal.h"

namespace fz {

// Update step of Lloyd's iterations.  The points are first grouped by the centre they were
// assigned to, each group in point order (integer work only: the grouping is the same in every
// run): sizes by a histogram, offsets by a scan, and one workgroup per centre that walks the
// assignment list and writes its members' ids in order (ballot / popcount compaction; the list is
// n ints and stays in L2).  Then one workgroup per (centre, 256 dimensions) adds up its members'
// rows in that order in fp64 and rounds the mean once to fp32, so the result does not depend on
// scheduling; every point row is read exactly once, in 1 KiB pieces.  A cluster without points keeps its centre.
// Histogram of the keys, up to kCountBins of them in LDS first (one global atomic per point and a few
// hundred addresses: 48 us for 50,000 points).
constexpr int kCountBins = 4096;
__global__ __launch_bounds__(256) void kmeans_count_kernel(const int32_t *assign, int64_t n, int64_t k, int32_t *sizes)
{
    __shared__ int hist[kCountBins];
    const int bins = (int)(k < kCountBins ? k : kCountBins);
    for (int c = threadIdx.x; c < bins; c += 256) hist[c] = 0;
    __syncthreads();
    const int64_t per = (n + gridDim.x - 1) / gridDim.x;
    const int64_t i1 = (blockIdx.x + 1) * per < n ? (blockIdx.x + 1) * per : n;
    for (int64_t i = blockIdx.x * per + threadIdx.x; i < i1; i += 256) {
        const int32_t c = assign[i];
        if (c >= 0 && c < bins)
            atomicAdd(&hist[c], 1);
        else if ((uint32_t)c < (uint64_t)k)
            atomicAdd(&sizes[c], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < bins; c += 256)
        if (hist[c]) atomicAdd(&sizes[c], hist[c]);
}

// offsets[c] = sizes[0] + .. + sizes[c-1], offsets[k] = total; one workgroup.  rank: the centres, the largest cluster
// first (up to 1,024 centres, else in order: it only spreads the update's work).
__global__ __launch_bounds__(1024) void kmeans_offsets_kernel(const int32_t *sizes, int64_t k, int32_t *offsets, int32_t *rank)
{
    __shared__ int size_s[1024];
    __shared__ int wave_tot[16];
    __shared__ int base_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) base_s = 0;
    __syncthreads();
    for (int64_t start = 0; start < k; start += 1024) {
        const int64_t c = start + tid;
        const int v = c < k ? sizes[c] : 0;
        int incl = v;   // inclusive scan within the wave
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        if (lane == 63) wave_tot[w] = incl;
        __syncthreads();
        int before = base_s;
        for (int i = 0; i < w; ++i) before += wave_tot[i];
        if (c < k) offsets[c] = before + incl - v;
        __syncthreads();
        if (tid == 1023) base_s = before + incl;
        __syncthreads();
    }
    if (tid == 0) offsets[k] = base_s;
    if (k <= 1024) {
        const int mine = tid < k ? sizes[tid] : 0;
        size_s[tid] = mine;
        __syncthreads();
        int larger = 0;
#pragma unroll 16
        for (int j = 0; j < (int)k; ++j) larger += (size_s[j] > mine) | ((size_s[j] == mine) & (j < tid));
        if (tid < k) rank[larger] = tid;
    } else {
        for (int64_t c = tid; c < k; c += 1024) rank[c] = (int32_t)c;
    }
}

// members[offsets[c] ..) = the ids of the points assigned to centre c = blockIdx.x, ascending.  Sixteen blocks of 1,024 points per
// step: bound by the latency of the list's reads and the barriers (50,000 points: one block a step 32 us,
// sixteen 22).
__global__ __launch_bounds__(1024) void kmeans_members_kernel(const int32_t *assign, int64_t n, const int32_t *offsets,
                                                              int32_t *members)
{
    constexpr int U = 16;
    __shared__ __attribute__((aligned(16))) int wave_tot[2][U * 16];
    const int c = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int base = offsets[c];
    if (offsets[c + 1] == base) return;   // uniform: an empty cluster
    int par = 0;
    for (int64_t start = 0; start < n; start += U * 1024, par ^= 1) {
        bool mine[U];
        uint64_t bal[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = start + u * 1024 + tid;
            mine[u] = i < n && assign[i] == c;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bal[u] = __ballot(mine[u]);
            if (lane == 0) wave_tot[par][u * 16 + w] = __builtin_popcountll(bal[u]);
        }
        __syncthreads();   // (two buffers: the next step's counts are written while slower waves still read these)
        // the 256 counts are in point order: lane l scans counts 4 l .. 4 l + 3
        const int4 c4 = reinterpret_cast<const int4 *>(wave_tot[par])[lane];
        const int sum = c4.x + c4.y + c4.z + c4.w;
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        // points before this wave's count of 1,024-point block u, which is count u * 16 + w: element w & 3 of lane (u * 16 + w) / 4
        const int mod = w & 3;
        const int before = incl - sum + (mod > 0 ? c4.x : 0) + (mod > 1 ? c4.y : 0) + (mod > 2 ? c4.z : 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int at = __builtin_amdgcn_readlane(before, u * 4 + (w >> 2));
            if (mine[u])
                members[base + at + __builtin_popcountll(bal[u] & ((1ull << lane) - 1ull))] = (int32_t)(start + u * 1024 + tid);
        }
        base += __builtin_amdgcn_readlane(incl, 63);
    }
}

// A workgroup per (centre, 256 dimensions) reads 64 rows' pieces of 1 KiB into registers, hands them on through LDS, and
// while the next 64 are on their way every thread adds up the 64 values of its dimension in order.  Clusters are uneven
// (50,000 x 8,192, 200 centres: the largest 1,862 points, half of them under 124), and a sum in point order cannot be
// shared out, so the largest decide when the kernel ends: with a wave per cluster and sixteen rows in flight their chains
// of loads took most of its 350 us.  Largest clusters first (rank): 290 us, 1.64 GB at 5.7 TB/s.
// VEC: rows start on 16-byte boundaries (d a multiple of 4).
typedef __attribute__((ext_vector_type(4))) float f32x4;
template <bool VEC>
__global__ __launch_bounds__(256) void kmeans_update_kernel(const float *points, const int32_t *offsets, const int32_t *members,
                                                            const int32_t *rank, int64_t k, int64_t d, const float *old_centers, float *new_centers)
{
    constexpr int U = 16;                     // rows per wave and batch
    __shared__ __attribute__((aligned(16))) float rows_s[4 * U][256];
    const int64_t place = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    if (place >= k) return;                   // uniform
    const int c = rank[place];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t dim0 = (int64_t)blockIdx.x * 256;
    const int m0 = offsets[c], m1 = offsets[c + 1];
    // the lane's four dimensions of a piece: consecutive, or 64 apart; past the row's end any will do
    int at[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int x = VEC ? lane * 4 + h : lane + 64 * h;
        at[h] = dim0 + x < d ? x : 0;
    }
    f32x4 v[U];
    auto load = [&](int j0) {                 // rows j0 + w U ..; past the end the last row again
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const int j = j0 + w * U + e;
            const float *src = points + (int64_t)members[j < m1 ? j : m1 - 1] * d + dim0;
            if constexpr (VEC) {
                v[e] = *reinterpret_cast<const f32x4 *>(src + at[0]);
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) v[e][h] = src[at[h]];
            }
        }
    };
    double acc = 0.0;
    if (m1 > m0) load(m0);
    for (int j0 = m0; j0 < m1; j0 += 4 * U) {
        __syncthreads();                      // the batch before has been added
#pragma unroll
        for (int e = 0; e < U; ++e) {
            if constexpr (VEC) {
                *reinterpret_cast<f32x4 *>(&rows_s[w * U + e][lane * 4]) = v[e];
            } else {
#pragma unroll
                for (int h = 0; h < 4; ++h) rows_s[w * U + e][lane + 64 * h] = v[e][h];
            }
        }
        __syncthreads();
        if (j0 + 4 * U < m1) load(j0 + 4 * U);
        const int cnt = m1 - j0 < 4 * U ? m1 - j0 : 4 * U;
        if (cnt == 4 * U) {
#pragma unroll 16
            for (int e = 0; e < 4 * U; ++e) acc += (double)rows_s[e][tid];   // in point order
        } else {
            for (int e = 0; e < cnt; ++e) acc += (double)rows_s[e][tid];
        }
    }
    const int64_t dim = dim0 + tid;
    if (dim < d) new_centers[(int64_t)c * d + dim] = m1 > m0 ? (float)(acc / (double)(m1 - m0)) : old_centers[(int64_t)c * d + dim];
}

// members = the ids 0 .. n-1 grouped by key (in [0, k)), each group ascending
static hipError_t launch_kmeans_group(const int32_t *key, int64_t n, int64_t k, int32_t *sizes, int32_t *offsets,
                                      int32_t *rank, int32_t *members, hipStream_t s)
{
    hipError_t e = launch_fill_i32(sizes, 0, k, s);
    if (e != hipSuccess) return e;
    const int64_t blocks = (n + 2047) / 2048 < 256 ? (n + 2047) / 2048 : 256;
    hipLaunchKernelGGL(kmeans_count_kernel, dim3((unsigned)blocks), dim3(256), 0, s, key, n, k, sizes);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(kmeans_offsets_kernel, dim3(1), dim3(1024), 0, s, sizes, k, offsets, rank);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(kmeans_members_kernel, dim3((unsigned)k), dim3(1024), 0, s, key, n, offsets, members);
    return hipGetLastError();
}

hipError_t launch_kmeans_update(const float *points, const int32_t *assign, int64_t n, int64_t d, int64_t k,
                                const float *old_centers, float *new_centers, int32_t *sizes, int32_t *offsets,
                                int32_t *rank, int32_t *members, hipStream_t s)
{
    hipError_t e = launch_kmeans_group(assign, n, k, sizes, offsets, rank, members, s);
    if (e != hipSuccess) return e;
    // (points, centres: 16-byte aligned by contract and by the workspace's layout)
    // (a cluster's workgroups in a row; in one dimension 4,097 centres of 2^20 values would be more than its 2^32 threads)
    const int64_t rows = k < 32768 ? k : 32768;
    const dim3 grid((unsigned)((d + 255) / 256), (unsigned)rows, (unsigned)((k + rows - 1) / rows));
    if (d % 4 == 0)
        hipLaunchKernelGGL(kmeans_update_kernel<true>, grid, dim3(256), 0, s, points, offsets, members, rank, k, d, old_centers, new_centers);
    else
        hipLaunchKernelGGL(kmeans_update_kernel<false>, grid, dim3(256), 0, s, points, offsets, members, rank, k, d, old_centers, new_centers);
    return hipGetLastError();
}

// Majority label (equal counts -> the smaller label), its share of the cluster, and the cluster
// size, one block per cluster, by a histogram of the members' labels in LDS (integer counts:
// no dependence on the order of the atomic additions).  An empty cluster gets label 0, share 0.
constexpr int kKmeansMaxClasses = 8192;

__global__ __launch_bounds__(1024) void kmeans_majority_kernel(const int32_t *assign, const int32_t *labels, int64_t n,
                                                               int num_classes, int32_t *majority, float *fraction,
                                                               int64_t *sizes)
{
    __shared__ int hist[kKmeansMaxClasses];
    __shared__ int best_s[16], bestl_s[16], size_s;
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int l = tid; l < num_classes; l += 1024) hist[l] = 0;
    if (tid == 0) size_s = 0;
    __syncthreads();
    int mine = 0;
    auto count = [&](int64_t i, int32_t a) {
        if (a != c) return;
        const int l = labels[i];
        if ((unsigned)l < (unsigned)num_classes) atomicAdd(&hist[l], 1);   // labels outside the contract are not counted
        ++mine;
    };
    int64_t i = tid;
    for (; i + 7 * 1024 < n; i += 8 * 1024) {   // eight loads in flight; most points belong to other clusters
        int32_t as[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) as[u] = assign[i + u * 1024];
#pragma unroll
        for (int u = 0; u < 8; ++u) count(i + u * 1024, as[u]);
    }
    for (; i < n; i += 1024) count(i, assign[i]);
    if (mine) atomicAdd(&size_s, mine);
    __syncthreads();
    int best = -1, bestl = 0;
    for (int l = tid; l < num_classes; l += 1024) {   // ascending l per thread: the first maximum is the smallest label
        if (hist[l] > best) {
            best = hist[l];
            bestl = l;
        }
    }
    auto better = [&](int b, int bl) {
        if (b > best || (b == best && bl < bestl)) {
            best = b;
            bestl = bl;
        }
    };
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const int b = __shfl_xor(best, off, 64), bl = __shfl_xor(bestl, off, 64);
        better(b, bl);
    }
    if (lane == 0) {
        best_s[w] = best;
        bestl_s[w] = bestl;
    }
    __syncthreads();
    if (tid == 0) {
        for (int t = 1; t < 16; ++t) better(best_s[t], bestl_s[t]);
        const int size = size_s;
        majority[c] = size ? bestl : 0;
        fraction[c] = size ? (float)((double)best / (double)size) : 0.f;
        if (sizes) sizes[c] = size;
    }
}

hipError_t launch_kmeans_majority(const int32_t *assign, const int32_t *labels, int64_t n, int num_classes, int64_t k,
                                  int32_t *majority, float *fraction, int64_t *sizes, hipStream_t s)
{
    if (num_classes < 1 || num_classes > kKmeansMaxClasses) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kmeans_majority_kernel, dim3((unsigned)k), dim3(1024), 0, s, assign, labels, n, num_classes,
                       majority, fraction, sizes);
    return hipGetLastError();
}

// dst[i] = src[i] for float arrays; rows of a [rows, d] matrix out of a [rows, d_pad] one
__global__ void copy_rows_f32_kernel(const float *src, int64_t src_stride, float *dst, int64_t rows, int64_t d)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows * d; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[(i / d) * src_stride + i % d];
}

hipError_t launch_copy_rows_f32(const float *src, int64_t src_stride, float *dst, int64_t rows, int64_t d, hipStream_t s)
{
    const int64_t total = rows * d;
    if (total <= 0) return hipSuccess;
    // (a grid of 2^32 threads and more is cut off without an error)
    const int64_t blocks = (total + 255) / 256 < (1 << 20) ? (total + 255) / 256 : 1 << 20;
    hipLaunchKernelGGL(copy_rows_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src, src_stride, dst, rows, d);
    return hipGetLastError();
}

__global__ void copy_i32_plain_kernel(const int32_t *src, int32_t *dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_copy_i32(const int32_t *src, int32_t *dst, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(copy_i32_plain_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

__global__ void fill_i32_kernel(int32_t *dst, int32_t v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = v;
}

hipError_t launch_fill_i32(int32_t *dst, int32_t v, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, v, n);
    return hipGetLastError();
}

}  // namespace fz
