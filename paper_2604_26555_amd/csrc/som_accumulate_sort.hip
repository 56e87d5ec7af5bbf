// Per-BMU sample sums and counts by counting sort:  S_k += x_i,  n_k += 1  for k = b_i  (the inner sums of Eq. 3).
//
// For rows wider than one feature window of the LDS kernels (som_accumulate_f64.hip: 63 features, one pass over all BMU
// indices and one strided pass over the rows per window, 64 launches at D = 2000), and for maps of many slabs
// (som_accumulate.hip, sort_pays).  Here the sample positions are sorted by
// node first, and then every row is read once, whole, by lanes that hold its node's running sum in registers (no atomics).
//   1. hist      a workgroup per block of samples counts its samples per node in LDS;
//   2. columns   per node, the counts of the blocks become running offsets, the total goes to n;
//   3. starts    the nodes' totals become start positions, and their samples are cut into segments;
//   4. scatter   every workgroup writes its samples' row numbers to their places;
//   5. sums      a group of lanes adds up a segment (four features a lane, float64) and stores it;
//   6. finish    a node's segments are added up in order.
// Bound by HBM in step 5 (D * 4 contiguous bytes per row); steps 1 to 4 cost about 25 us at 10^6 samples.  (With equal ranges of
// the sorted order and an atomic per feature at every node boundary instead of segments, step 5 took 217 us at 10^5 x 2000.)
// The order of a node's samples within a block is not fixed, so a sum can differ in its last bits between runs (float64).
//
// Fixed order of summation (som_set_reproducible): the same with a stable sort: a block is one wavefront's, which ranks its 64
// samples at a time by ballots, one for each bit of the nodes' numbers.
#include "som_internal.hpp"

namespace som {

constexpr int kSortThreads = 1024;
constexpr int kSortNodes = 16384;         // per-node counters of a workgroup in LDS (64 KB)
constexpr int kSortBlocks = 512;          // blocks of samples at most
constexpr int kStableWaves = 4;           // wavefronts (blocks) of a workgroup of the stable sort
constexpr int kStableBlocks = 1024;
constexpr int kStableNodes = 8192;        // per-node counters of four wavefronts in LDS (128 KB)

__global__ void __launch_bounds__(kSortThreads) sort_hist_kernel(const int32_t* __restrict__ bmu, int64_t m, int K, int64_t per_block,
                                                                 uint32_t* __restrict__ hist)
{
    extern __shared__ uint32_t sort_lds[];
    const int tid = threadIdx.x;
    for (int k = tid; k < K; k += kSortThreads) sort_lds[k] = 0u;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * per_block, hi = lo + per_block < m ? lo + per_block : m;
    for (int64_t i = lo + tid; i < hi; i += kSortThreads) {
        const int b = bmu[i];
        if (b >= 0 && b < K) atomicAdd(&sort_lds[b], 1u);
    }
    __syncthreads();
    for (int k = tid; k < K; k += kSortThreads) hist[(size_t)blockIdx.x * K + k] = sort_lds[k];
}

// hist[block][k] -> number of node k's samples in the blocks before; total[k]; n[k] (+)= total[k].  NODES nodes and
// 1024 / NODES runs of blocks per workgroup.  Small maps wait for latency: a thread's loads follow each other, so that short runs count
// (64 nodes and sixteen runs: 12.6 us for 1023 blocks of 400 nodes, 6.0 with 16 nodes).  Of large ones the counts are tens of MB, and 16
// nodes are half a line: the stable sum of 300,000 rows of 10 on 8000 nodes 155 us, 137 with 32 nodes; 500,000 of 20 on 2304
// nodes 94.8 and 92.4.
template <int NODES>
__global__ void __launch_bounds__(1024) sort_columns_kernel(uint32_t* __restrict__ hist, int K, int blocks, uint32_t* __restrict__ total,
                                                            unsigned long long* __restrict__ n, int zero_first)
{
    __shared__ uint32_t run[16][NODES];
    constexpr int kRuns = 1024 / NODES;
    const int l = threadIdx.x & (NODES - 1), seg = threadIdx.x / NODES, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * NODES + l, kc = k < K ? k : K - 1;
    const int per = (blocks + kRuns - 1) / kRuns, lo = seg * per, hi = lo + per < blocks ? lo + per : blocks;
    uint32_t s = 0u;
    for (int b0 = lo; b0 < hi; b0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)(b0 + u < hi ? b0 + u : lo) * K + kc];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += b0 + u < hi ? v[u] : 0u;
    }
    uint32_t at = s;                                           // up to and with this run, among the wavefront's
#pragma unroll
    for (int o = NODES; o < 64; o <<= 1) {
        const uint32_t before = __shfl_up(at, o);
        if (lane >= o) at += before;
    }
    if (lane >= 64 - NODES) run[wave][l] = at;
    at -= s;
    __syncthreads();
    uint32_t all = 0u;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const uint32_t v = run[q][l];
        at += q < wave ? v : 0u;
        all += v;
    }
    if (k >= K) return;
    for (int b0 = lo; b0 < hi; b0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = hist[(size_t)(b0 + u < hi ? b0 + u : lo) * K + k];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (b0 + u < hi) {
                hist[(size_t)(b0 + u) * K + k] = at;
                at += v[u];
            }
        }
    }
    if (seg == 0) {
        total[k] = all;
        n[k] = (zero_first ? 0ull : n[k]) + all;
    }
}

// row numbers to their places: start[k] + what the blocks before hold of node k + a place inside the block
__global__ void __launch_bounds__(kSortThreads) sort_scatter_kernel(const int32_t* __restrict__ bmu, const uint32_t* __restrict__ idx,
                                                                    int64_t m, int K, int64_t per_block,
                                                                    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ start,
                                                                    uint32_t* __restrict__ perm)
{
    extern __shared__ uint32_t sort_lds[];
    const int tid = threadIdx.x;
    for (int k = tid; k < K; k += kSortThreads) sort_lds[k] = start[k] + hist[(size_t)blockIdx.x * K + k];
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * per_block, hi = lo + per_block < m ? lo + per_block : m;
    for (int64_t i = lo + tid; i < hi; i += kSortThreads) {
        const int b = bmu[i];
        if (b >= 0 && b < K) perm[atomicAdd(&sort_lds[b], 1u)] = idx ? idx[i] : (uint32_t)i;
    }
}

// The stable sort's histogram and scatter: a block is a wavefront's.
__global__ void __launch_bounds__(64 * kStableWaves) stable_hist_kernel(const int32_t* __restrict__ bmu, int64_t m, int K, int64_t per_block,
                                                                        int blocks, uint32_t* __restrict__ hist)
{
    extern __shared__ uint32_t sort_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int block = blockIdx.x * kStableWaves + wave;
    uint32_t* count = sort_lds + wave * K;
    for (int k = lane; k < K; k += 64) count[k] = 0u;
    __builtin_amdgcn_wave_barrier();
    if (block >= blocks) return;                              // (no barrier below)
    const int64_t lo = (int64_t)block * per_block, hi = lo + per_block < m ? lo + per_block : m;
    for (int64_t i = lo + lane; i < hi; i += 64) {
        const int b = bmu[i];
        if (b >= 0 && b < K) atomicAdd(&count[b], 1u);
    }
    __builtin_amdgcn_wave_barrier();
    for (int k = lane; k < K; k += 64) hist[(size_t)block * K + k] = count[k];
}

// exclusive scan over the nodes: start[k] of the totals and seg[k] of the segments of `rows` samples (K + 1 entries each)
__global__ void __launch_bounds__(1024) sort_starts_kernel(const uint32_t* __restrict__ total, int K, uint32_t rows,
                                                             uint32_t* __restrict__ start, uint32_t* __restrict__ seg)
{
    __shared__ uint2 wave_sum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (K + 1023) / 1024, k0 = tid * per;
    uint2 mine = make_uint2(0u, 0u);
    for (int u = 0; u < per; ++u) {
        const uint32_t t = k0 + u < K ? total[k0 + u] : 0u;
        mine.x += t;
        mine.y += (t + rows - 1) / rows;
    }
    uint2 incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(incl.x, o), y = __shfl_up(incl.y, o);
        if (lane >= o) {
            incl.x += x;
            incl.y += y;
        }
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    uint2 at = make_uint2(incl.x - mine.x, incl.y - mine.y);
    for (int w = 0; w < wave; ++w) {
        at.x += wave_sum[w].x;
        at.y += wave_sum[w].y;
    }
    for (int u = 0; u < per && k0 + u < K; ++u) {
        const uint32_t t = total[k0 + u];
        start[k0 + u] = at.x;
        seg[k0 + u] = at.y;
        at.x += t;
        at.y += (t + rows - 1) / rows;
        if (k0 + u == K - 1) {
            start[K] = at.x;
            seg[K] = at.y;
        }
    }
}

__global__ void __launch_bounds__(64 * kStableWaves) stable_scatter_kernel(const int32_t* __restrict__ bmu, const uint32_t* __restrict__ idx,
                                                                           int64_t m, int K, int64_t per_block, int blocks,
                                                                           const uint32_t* __restrict__ hist,
                                                                           const uint32_t* __restrict__ start, uint32_t* __restrict__ perm)
{
    extern __shared__ uint32_t sort_lds[];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int block = blockIdx.x * kStableWaves + wave;
    if (block >= blocks) return;                              // (no barrier: a wavefront works on its own)
    uint32_t* place = sort_lds + wave * K;
    for (int k = lane; k < K; k += 64) place[k] = start[k] + hist[(size_t)block * K + k];
    __builtin_amdgcn_wave_barrier();
    const int64_t lo = (int64_t)block * per_block, hi = lo + per_block < m ? lo + per_block : m;
    const int bits = 32 - __builtin_clz((unsigned)K);
    int b_next = lo + lane < hi ? bmu[lo + lane] : -1;
    for (int64_t i0 = lo; i0 < hi; i0 += 64) {
        const int64_t i = i0 + lane;
        int b = b_next;
        b_next = i + 64 < hi ? bmu[i + 64] : -1;
        if (b >= K) b = -1;
        const uint32_t base = b >= 0 ? place[b] : 0u;
        // rank of every lane among the lanes of the same node, in lane order: whose numbers agree in every bit (a round for each node that the
        // wavefront has took three quarters of the kernel: 500,000 samples of 400 nodes 25.8 us, 9.8 this way)
        unsigned long long peers = __ballot(b >= 0);
        for (int bit = 0; bit < bits; ++bit) {
            const bool on = (b >> bit & 1) != 0;
            const unsigned long long m_on = __ballot(on);
            peers &= on ? m_on : ~m_on;
        }
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi((unsigned)(peers >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)peers, 0));
        const uint32_t same = (uint32_t)__popcll(peers);
        __builtin_amdgcn_wave_barrier();
        if (b >= 0) {
            perm[base + rank] = idx ? idx[i] : (uint32_t)i;
            if (rank == 0u) place[b] = base + same;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// LANES lanes per segment of one node's samples, four features a lane (slab: 4 LANES features); the sums go to
// part[seg], added up by sort_finish_kernel, or to S (null: S is added to) where the node has no other segment
template <int LANES>
__global__ void __launch_bounds__(256) sort_sums_kernel(const float* __restrict__ X, int D, int64_t ldx, const uint32_t* __restrict__ start,
                                                          const uint32_t* __restrict__ seg, int K, const uint32_t* __restrict__ perm,
                                                          uint32_t rows, int slabs, double* part, double* S)
{
    constexpr int per_group = 256 / LANES;
    const int sub = threadIdx.x % LANES, first_lane = (threadIdx.x & 63) - sub;
    const int64_t units = (int64_t)gridDim.x * per_group;
    const int64_t all = (int64_t)seg[K] * slabs;
    for (int64_t unit = (int64_t)blockIdx.x * per_group + threadIdx.x / LANES; unit < all; unit += units) {
        const int slab = (int)(unit % slabs);
        const uint32_t sg = (uint32_t)(unit / slabs);
        int k = 0, top = K;                                   // the last node with seg[k] <= sg
        while (top - k > 1) {
            const int mid = (k + top) >> 1;
            if (seg[mid] <= sg) k = mid;
            else top = mid;
        }
        const uint32_t lo = start[k] + (sg - seg[k]) * rows, end = start[k + 1];
        const uint32_t hi = end - lo < rows ? end : lo + rows;
        const int f_own = (slab * LANES + sub) * 4;
        const bool on = f_own < D;
        const int f = f_own < D - 4 ? f_own : D - 4, shift = f_own - f;
        double* const to = (S && seg[k + 1] - seg[k] == 1) ? S + (size_t)k * D : part + (size_t)sg * D;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        // G rows in hand and as many under way, and the numbers of those behind: 10^6 x 200 171 us, 10^5 x 2000 168, where a plain read of X takes
        // 157.  (Numbers and rows of each eight waited for in turn: 222 and 207; sixteen at a time 250.)  Sixteen lanes have four rows to an
        // instruction and short segments: 10^6 x 50 on 4096 nodes 54 us whether four or eight.
        constexpr int G = LANES == 16 ? 8 : 4;
        auto numbers = [&](uint32_t p) {
            const int left = hi - p < (uint32_t)G ? (int)(hi - p) : G;
            return perm[p + (sub < left ? sub : left - 1)];
        };
        auto load = [&](uint32_t p, uint32_t row_mine, float4 (&v)[G]) {
            const int left = hi - p < (uint32_t)G ? (int)(hi - p) : G;
#pragma unroll
            for (int u = 0; u < G; ++u) {
                const uint32_t row = __shfl(row_mine, first_lane + (u < left ? u : 0));
                if (u < left && on) __builtin_memcpy(&v[u], X + (int64_t)row * ldx + f, sizeof(float4));
                else v[u] = float4{0.f, 0.f, 0.f, 0.f};
            }
        };
        auto add = [&](const float4 (&v)[G]) {
#pragma unroll
            for (int u = 0; u < G; ++u) {
                acc[0] += (double)v[u].x;
                acc[1] += (double)v[u].y;
                acc[2] += (double)v[u].z;
                acc[3] += (double)v[u].w;
            }
        };
        float4 one[G], two[G];
        uint32_t row_next = numbers(lo + G < hi ? lo + G : lo);
        load(lo, numbers(lo), one);
        for (uint32_t p = lo;; p += 2 * G) {
            const uint32_t row_one = numbers(p + 2 * G < hi ? p + 2 * G : p);
            if (p + G < hi) load(p + G, row_next, two);
            add(one);
            if (p + G >= hi) break;
            row_next = numbers(p + 3 * G < hi ? p + 3 * G : p);
            if (p + 2 * G < hi) load(p + 2 * G, row_one, one);
            add(two);
            if (p + 2 * G >= hi) break;
        }
        if (on) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (t >= shift) to[f + t] = acc[t];
        }
    }
}

// a workgroup per node, 64 features at a time: a run of the node's segments per wavefront, added up in order (a single segment's
// sums are in S already; with a workgroup per 64 features their mere launch took 60 us at D = 2000).  Sixteen loads under way in
// a run, and eight runs, four where the workgroups are many and walk on: sixteen runs, four loads at a time, kept the chip in
// wavefronts without a segment (K = 1024, D = 2000: 58 us, 21 now; D = 200: 16.7, 11; K = 4096, D = 50: 26.5, 21).  What is left is the
// chain of a node with many segments, so up to eight workgroups share its features (`shares`): the whole call with half of 50,000 rows x
// 1000 on one of 1024 nodes 88 us with sixteen runs, 103 with four and four workgroups, 86 with eight; evenly spread rows 76, 64, 65.
__global__ void __launch_bounds__(1024) sort_finish_kernel(const double* __restrict__ part, const uint32_t* __restrict__ seg, int D,
                                                             int zero_first, double* __restrict__ S)
{
    __shared__ double run[16][64];
    const int l = threadIdx.x & 63, r = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = blockIdx.x;
    const uint32_t first = seg[k], all = seg[k + 1] - first, runs = blockDim.x >> 6, per = (all + runs - 1) / runs;
    if (all == 1 && zero_first) return;
    const uint32_t lo = r * per, hi = lo + per < all ? lo + per : all;
    for (int f0 = 64 * blockIdx.y; f0 < D; f0 += 64 * gridDim.y) {
        const int f = f0 + l;
        double s = 0.0;
        const int fc = f < D ? f : D - 1;
        for (uint32_t q0 = lo; q0 < hi; q0 += 16) {
            double v[16];
#pragma unroll
            for (uint32_t u = 0; u < 16; ++u) {
                v[u] = 0.0;
                if (q0 + u < hi) v[u] = part[(size_t)(first + q0 + u) * D + fc];
            }
#pragma unroll
            for (uint32_t u = 0; u < 16; ++u) s += v[u];
        }
        run[r][l] = s;
        __syncthreads();
        if (r == 0 && f < D) {
#pragma unroll
            for (uint32_t q = 1; q < 16; ++q) s += q < runs ? run[q][l] : 0.0;
            const size_t e = (size_t)k * D + f;
            S[e] = (zero_first ? 0.0 : S[e]) + s;
        }
        __syncthreads();
    }
}

static int sort_workspace(som_ctx* ctx, size_t need)
{
    if (need <= ctx->acc_bytes) return SOM_OK;
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
    return SOM_OK;
}

// Returns 1 when the shape is not served by this path, SOM_OK on success, a negative code on failure.
int accumulate_sort_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, const int32_t* bmu,
                        int32_t K, double* S, unsigned long long* n, bool zero_first, bool stable)
{
    if (m <= 0 || D < 4 || K > (stable ? kStableNodes : kSortNodes)) return 1;
    const int most = stable ? kStableBlocks : kSortBlocks;
    int64_t per_block = (m + most - 1) / most;
    if (per_block < (stable ? 256 : 2048)) per_block = stable ? 256 : 2048;
    const int blocks = (int)((m + per_block - 1) / per_block);
    // segments: about four wavefronts per SIMD, 32 to 1024 rows (half as long: 213 -> 276 us at 10^6 x 200)
    const int lanes = D <= 64 ? 16 : D <= 128 ? 32 : 64;
    const int slabs = (D + 4 * lanes - 1) / (4 * lanes);
    int64_t rows = m * lanes * slabs / (256 * 4 * 4 * 64);
    if (slabs > 1) rows /= 2;                 // (10^5 x 2000: 2.33, 2.13, 2.07 ms an epoch with 390, 195, 97 rows)
    // Every wavefront reads its own stretch of X.  Where X is large and the nodes' shares are uneven, long segments lose a third
    // or more at some lengths (K = 1024, 150 features: 5 * 10^6 rows 1365 us with 1024 rows, 922 with 256; 10^7 rows of 72
    // features 1472, 994; K = 4096: 1520, 1131), and even ones of 256 rows 5 % at most (K = 100, 10^7 rows of 150: 1692, 1761).
    const int64_t longest = (double)m * D * 4.0 > 2.5e9 ? 256 : 1024;
    rows = rows < 32 ? 32 : rows > longest ? longest : rows;
    const size_t segs_most = (size_t)(m / rows) + K;
    const size_t hist_words = (size_t)blocks * K, words = (hist_words + 3 * (size_t)K + 2 + (size_t)m + 1) / 2 * 2;
    if (int rc = sort_workspace(ctx, words * sizeof(uint32_t) + segs_most * D * sizeof(double))) return rc;
    uint32_t* hist = (uint32_t*)ctx->acc_blob;
    uint32_t* total = hist + hist_words;
    uint32_t* start = total + K;
    uint32_t* seg = start + K + 1;
    uint32_t* perm = seg + K + 1;
    double* part = (double*)(hist + words);
    const size_t lds = (size_t)K * sizeof(uint32_t) * (stable ? kStableWaves : 1);
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    if (!attr_set) {
        for (const void* k : {reinterpret_cast<const void*>(stable_hist_kernel), reinterpret_cast<const void*>(stable_scatter_kernel),
                              reinterpret_cast<const void*>(sort_hist_kernel), reinterpret_cast<const void*>(sort_scatter_kernel)})
            if (int rc = check_hip(ctx, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kStableNodes * kStableWaves * 4),
                                   "raising the dynamic LDS limit"))
                return rc;
        attr_set = true;
    }
    const dim3 grid(stable ? (blocks + kStableWaves - 1) / kStableWaves : blocks), wg(stable ? 64 * kStableWaves : kSortThreads);
    if (stable) hipLaunchKernelGGL(stable_hist_kernel, grid, wg, lds, ctx->stream, bmu, m, K, per_block, blocks, hist);
    else hipLaunchKernelGGL(sort_hist_kernel, grid, wg, lds, ctx->stream, bmu, m, K, per_block, hist);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) histogram launch")) return rc;
    const int columns = K < 2048 ? 16 : 32;                 // (timed at K = 1600, 2025, 2304 and above)
    hipLaunchKernelGGL(columns == 16 ? sort_columns_kernel<16> : sort_columns_kernel<32>, dim3((K + columns - 1) / columns), dim3(1024), 0, ctx->stream, hist, K, blocks, total, n, zero_first ? 1 : 0);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) offsets launch")) return rc;
    hipLaunchKernelGGL(sort_starts_kernel, dim3(1), dim3(1024), 0, ctx->stream, total, K, (uint32_t)rows, start, seg);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) starts launch")) return rc;
    if (stable) hipLaunchKernelGGL(stable_scatter_kernel, grid, wg, lds, ctx->stream, bmu, idx, m, K, per_block, blocks, hist, start, perm);
    else hipLaunchKernelGGL(sort_scatter_kernel, grid, wg, lds, ctx->stream, bmu, idx, m, K, per_block, hist, start, perm);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) scatter launch")) return rc;
    const int64_t groups_most = ((int64_t)segs_most * slabs * lanes + 255) / 256;
    const unsigned groups = (unsigned)(groups_most < 8192 ? groups_most : 8192);
    auto kern = lanes == 16 ? sort_sums_kernel<16> : lanes == 32 ? sort_sums_kernel<32> : sort_sums_kernel<64>;
    hipLaunchKernelGGL(kern, dim3(groups), dim3(256), 0, ctx->stream, X, D, ldx, start, seg, K, perm, (uint32_t)rows, slabs, part,
                       zero_first ? S : (double*)nullptr);
    if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (sort) sums launch")) return rc;
    // D > 256: workgroups of a node, which share its features (K = 4096, D = 600: 49.5 us a call with four, 52.4 with eight)
    const int most_shares = K <= 2048 ? 8 : 4, shares = D <= 256 ? 1 : (D + 63) / 64 < most_shares ? (D + 63) / 64 : most_shares;
    hipLaunchKernelGGL(sort_finish_kernel, dim3(K, shares), dim3(D > 256 ? 256 : 512), 0, ctx->stream, part, seg, D, zero_first ? 1 : 0, S);
    return check_hip(ctx, hipGetLastError(), "accumulate (sort) finish launch");
}

} // namespace som
