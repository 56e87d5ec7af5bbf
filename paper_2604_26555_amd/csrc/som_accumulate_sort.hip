// Per-BMU sample sums and counts by counting sort:  S_k += x_i,  n_k += 1  for k = b_i  (the inner sums of Eq. 3).
//
// For rows wider than one feature window of the LDS kernels (som_accumulate_f64.hip: 63 features, one pass over all BMU
// indices and one strided pass over the rows per window, 32 launches at D = 2000).  Here the sample positions are sorted by
// node first, and then every row is read once, whole, by the wavefront that holds its node's running sum in registers:
// no atomics but one per feature where a range of the sorted order begins or ends inside a node's samples.
//   1. hist      a workgroup per block of samples counts its samples per node in LDS (and clears S where asked);
//   2. columns   per node, the counts of the blocks become running offsets, the total goes to n;
//   3. scatter   every workgroup adds up the nodes' totals to start positions and writes its samples' row numbers there;
//   4. sums      lane groups take equal ranges of the sorted order.
// Bound by HBM in step 4 (D * 4 contiguous bytes per row); steps 1 to 3 cost about 20 us at 10^6 samples.
// The order of a node's samples within a block is not fixed, so a sum can differ in its last bits between runs (float64).
#include "som_internal.hpp"

#include <hip/amd_detail/amd_hip_unsafe_atomics.h>

namespace som {

constexpr int kSortThreads = 1024;
constexpr int kSortNodes = 16384;         // per-node counters of a workgroup in LDS (64 KB)
constexpr int kSortBlocks = 512;          // blocks of samples at most

__global__ void __launch_bounds__(kSortThreads) sort_hist_kernel(const int32_t* __restrict__ bmu, int64_t m, int K, int64_t per_block,
                                                                 uint32_t* __restrict__ hist, double* __restrict__ S_clear,
                                                                 size_t cells)
{
    extern __shared__ uint32_t sort_lds[];
    const int tid = threadIdx.x;
    for (int k = tid; k < K; k += kSortThreads) sort_lds[k] = 0u;
    if (S_clear)
        for (size_t c = (size_t)blockIdx.x * kSortThreads + tid; c < cells; c += (size_t)gridDim.x * kSortThreads) S_clear[c] = 0.0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * per_block, hi = lo + per_block < m ? lo + per_block : m;
    for (int64_t i = lo + tid; i < hi; i += kSortThreads) {
        const int b = bmu[i];
        if (b >= 0 && b < K) atomicAdd(&sort_lds[b], 1u);
    }
    __syncthreads();
    for (int k = tid; k < K; k += kSortThreads) hist[(size_t)blockIdx.x * K + k] = sort_lds[k];
}

// hist[block][k] -> number of node k's samples in the blocks before; total[k]; n[k] (+)= total[k].  64 nodes and sixteen
// runs of blocks per workgroup.
__global__ void __launch_bounds__(1024) sort_columns_kernel(uint32_t* __restrict__ hist, int K, int blocks, uint32_t* __restrict__ total,
                                                            unsigned long long* __restrict__ n, int zero_first)
{
    __shared__ uint32_t run[16][64];
    const int l = threadIdx.x & 63, seg = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + l;
    const int per = (blocks + 15) / 16, lo = seg * per, hi = lo + per < blocks ? lo + per : blocks;
    uint32_t s = 0u;
    if (k < K) {
#pragma unroll 8
        for (int b = lo; b < hi; ++b) s += hist[(size_t)b * K + k];
    }
    run[seg][l] = s;
    __syncthreads();
    if (k >= K) return;
    uint32_t at = 0u, all = 0u;
    for (int q = 0; q < 16; ++q) {
        const uint32_t v = run[q][l];
        at += q < seg ? v : 0u;
        all += v;
    }
    for (int b0 = lo; b0 < hi; b0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = b0 + u < hi ? hist[(size_t)(b0 + u) * K + k] : 0u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (b0 + u < hi) hist[(size_t)(b0 + u) * K + k] = at;
            at += v[u];
        }
    }
    if (seg == 0) {
        total[k] = all;
        n[k] = (zero_first ? 0ull : n[k]) + all;
    }
}

// start[k] = samples of the nodes before k (k = 0 .. K); row numbers to their places.  Workgroup 0 also writes start.
__global__ void __launch_bounds__(kSortThreads) sort_scatter_kernel(const int32_t* __restrict__ bmu, const uint32_t* __restrict__ idx,
                                                                    int64_t m, int K, int64_t per_block,
                                                                    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ total,
                                                                    uint32_t* __restrict__ start, uint32_t* __restrict__ perm)
{
    extern __shared__ uint32_t sort_lds[];
    __shared__ uint32_t wave_sum[kSortThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // exclusive scan of the totals: thread t takes K / 1024 consecutive nodes
    const int per = (K + kSortThreads - 1) / kSortThreads, k0 = tid * per;
    uint32_t mine = 0u;
    for (int u = 0; u < per; ++u) mine += k0 + u < K ? total[k0 + u] : 0u;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    for (int u = 0; u < per; ++u) {
        const int k = k0 + u;
        if (k >= K) break;
        if (blockIdx.x == 0) {
            start[k] = at;
            if (k == K - 1) start[K] = at + total[k];
        }
        sort_lds[k] = at + hist[(size_t)blockIdx.x * K + k];
        at += total[k];
    }
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * per_block, hi = lo + per_block < m ? lo + per_block : m;
    for (int64_t i = lo + tid; i < hi; i += kSortThreads) {
        const int b = bmu[i];
        if (b >= 0 && b < K) perm[atomicAdd(&sort_lds[b], 1u)] = idx ? idx[i] : (uint32_t)i;
    }
}

// LANES lanes (32 or 64) per range of the sorted order, four features a lane, features [4 LANES slab, ...) of the row.
template <int LANES>
__global__ void __launch_bounds__(256) sort_sums_kernel(const float* __restrict__ X, int D, int64_t ldx, const uint32_t* __restrict__ start,
                                                        int K, const uint32_t* __restrict__ perm, int per_range, int slabs,
                                                        double* __restrict__ S)
{
    constexpr int per_group = 256 / LANES;
    const int sub = threadIdx.x % LANES, first_lane = (threadIdx.x & 63) - sub;
    const int64_t unit = (int64_t)blockIdx.x * per_group + threadIdx.x / LANES;
    const int slab = (int)(unit % slabs);
    const int64_t range = unit / slabs;
    const uint32_t all = start[K];
    const int64_t lo = range * per_range;
    const bool work = lo < (int64_t)all;
    const int64_t hi = lo + per_range < (int64_t)all ? lo + per_range : (int64_t)all;
    // node of position lo: the last k with start[k] <= lo
    int k = 0;
    if (work) {
        int top = K;
        while (top - k > 1) {
            const int mid = (k + top) >> 1;
            if ((int64_t)start[mid] <= lo) k = mid;
            else top = mid;
        }
    }
    // this lane's four features: a window [f, f + 4) inside the row, its leading elements another lane's where it is shifted back
    const int f_own = (slab * LANES + sub) * 4;
    const bool on = f_own < D;
    const int f = f_own < D - 4 ? f_own : D - 4, shift = f_own - f;
    int64_t next = work ? (int64_t)start[k + 1] : 0;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    auto flush = [&]() {
        if (on) {
            double* s = S + (size_t)k * D + f;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t >= shift) unsafeAtomicAdd(&s[t], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = 0.0;
    };
    constexpr int G = 8;                            // rows in flight
    if (work)
        for (int64_t p = lo; p < hi;) {
            while (p >= next) {                    // (empty nodes in between)
                if (p > lo) flush();
                ++k;
                next = (int64_t)start[k + 1];
            }
            const int64_t stop = next < hi ? next : hi;
            // row numbers of up to G rows at a time, one per lane, handed round
            const int left = stop - p < G ? (int)(stop - p) : G;
            const uint32_t row_mine = perm[p + (sub < left ? sub : left - 1)];
            float4 v[G];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const uint32_t row = __shfl(row_mine, first_lane + (u < left ? u : 0));
                if (u < left && on) __builtin_memcpy(&v[u], X + (int64_t)row * ldx + f, sizeof(float4));
                else v[u] = float4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < G; ++u) {
                acc[0] += (double)v[u].x;
                acc[1] += (double)v[u].y;
                acc[2] += (double)v[u].z;
                acc[3] += (double)v[u].w;
            }
            p += left;
            if (p >= hi) flush();
        }
}

// Returns 1 when the shape is not served by this path, SOM_OK on success, a negative code on failure.
int accumulate_sort_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, const int32_t* bmu,
                        int32_t K, double* S, unsigned long long* n, bool zero_first)
{
    if (m <= 0 || D < 4 || K > kSortNodes) return 1;
    int64_t per_block = (m + kSortBlocks - 1) / kSortBlocks;
    if (per_block < 2048) per_block = 2048;
    const int blocks = (int)((m + per_block - 1) / per_block);
    const size_t hist_words = (size_t)blocks * K, small_words = 2 * (size_t)K + 1;
    const size_t need = (hist_words + small_words + (size_t)m) * sizeof(uint32_t);
    if (need > ctx->acc_bytes) {
        if (ctx->acc_blob) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->acc_blob);
            ctx->acc_blob = nullptr;
            ctx->acc_bytes = 0;
        }
        if (hipMalloc(&ctx->acc_blob, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the accumulation workspace", need);
        }
        ctx->acc_bytes = need;
    }
    uint32_t* hist = (uint32_t*)ctx->acc_blob;
    uint32_t* total = hist + hist_words;
    uint32_t* start = total + K;
    uint32_t* perm = start + K + 1;
    const size_t lds = (size_t)K * sizeof(uint32_t);
    hipLaunchKernelGGL(sort_hist_kernel, dim3(blocks), dim3(kSortThreads), lds, ctx->stream, bmu, m, K, per_block, hist,
                       zero_first ? S : (double*)nullptr, (size_t)K * D);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) histogram launch")) return rc;
    hipLaunchKernelGGL(sort_columns_kernel, dim3((K + 63) / 64), dim3(1024), 0, ctx->stream, hist, K, blocks, total, n, zero_first ? 1 : 0);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) offsets launch")) return rc;
    hipLaunchKernelGGL(sort_scatter_kernel, dim3(blocks), dim3(kSortThreads), lds, ctx->stream, bmu, idx, m, K, per_block, hist, total,
                       start, perm);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) scatter launch")) return rc;
    // Ranges: about eight wavefronts per SIMD over the slabs, but no shorter than 32 rows (the additions at a range's two
    // ends are atomics on S).
    const int lanes = D <= 128 ? 32 : 64;
    const int slabs = (D + 4 * lanes - 1) / (4 * lanes);
    int64_t ranges = (int64_t)256 * 4 * 8 * (64 / lanes) / slabs;
    if (ranges < 1) ranges = 1;
    int64_t per_range = (m + ranges - 1) / ranges;
    if (per_range < 32) per_range = 32;
    ranges = (m + per_range - 1) / per_range;
    const int64_t groups = (ranges * slabs * lanes + 255) / 256;
    if (lanes == 32)
        hipLaunchKernelGGL(sort_sums_kernel<32>, dim3((unsigned)groups), dim3(256), 0, ctx->stream, X, D, ldx, start, K, perm,
                           (int)per_range, slabs, S);
    else
        hipLaunchKernelGGL(sort_sums_kernel<64>, dim3((unsigned)groups), dim3(256), 0, ctx->stream, X, D, ldx, start, K, perm,
                           (int)per_range, slabs, S);
    return check_hip(ctx, hipGetLastError(), "accumulate (sort) sums launch");
}

} // namespace som
