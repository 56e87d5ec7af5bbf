// Data-driven neighbourhood graphs on the GPU (paper Sections 3.2.1-3.2.2, Algorithms 1 and 2):
//   pairwise squared node distances  ->  edge set (minimum spanning tree, or relative neighbourhood graph by the
//   blocker test)  ->  adjacency lists  ->  all-pairs hop counts G (float32, +inf where unreachable).
// Everything that decides an edge is float64 and uses direct differences, so the graphs agree with a float64
// host construction except on exact ties.  Work per rebuild at K = 1024: K^2 D distance flops, K^3 (max, min)
// operations for the blocker test, K breadth-first searches.
//   node_d2_kernel     d2[p][q] = sum_d (w_pd - w_qd)^2
//   boruvka_*          spanning tree for K <= 4096: <= log2 K rounds of (cheapest outgoing edge per node over all
//                      compute units, per-component minimum + merge in one workgroup)
//   mst_prim_kernel    spanning tree for larger K: Prim's method in one workgroup, K rounds of (arg-min, key update)
//   rng_near / rng_prefilter / rng_verify   pair (p, q) survives unless some r has max(d2[p][r], d2[q][r]) <
//                      d2[p][q]: every pair against 64 nodes near p first, the few pairs left against all nodes
//   csr_*              degree count, exclusive scan, ascending neighbour lists
//   bfs_kernel         one wavefront per source, frontier queue and distance row in LDS
//   tree_tour_kernel, tree_hops_kernel   the same for spanning trees: the nodes in depth-first order with their depths, and minima of those
#include "som_internal.hpp"

#include <math.h>

namespace som {

constexpr int kBoruvkaMaxNodes = 4096;   // 24 bytes of LDS per node in the merge kernel

// 32 x 32 pairs per workgroup, features staged through LDS 32 at a time; every pair sums over d in ascending order
__global__ void __launch_bounds__(256) node_d2_kernel(const float* __restrict__ W, int K, int D, double* __restrict__ d2)
{
    __shared__ float Wp[32][33];
    __shared__ float Wq[32][33];
    const int tid = threadIdx.x;
    const int p0 = blockIdx.x * 32, q0 = blockIdx.y * 32;
    const int pi = tid >> 5, qi = tid & 31;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    for (int d0 = 0; d0 < D; d0 += 32) {
        __syncthreads();
        for (int e = tid; e < 32 * 32; e += 256) {
            const int i = e >> 5, dd = e & 31;
            const bool in = d0 + dd < D;
            Wp[i][dd] = (in && p0 + i < K) ? W[(size_t)(p0 + i) * D + d0 + dd] : 0.0f;
            Wq[i][dd] = (in && q0 + i < K) ? W[(size_t)(q0 + i) * D + d0 + dd] : 0.0f;
        }
        __syncthreads();
        const int lim = (D - d0 < 32) ? D - d0 : 32;
        for (int dd = 0; dd < lim; ++dd) {
            const double b = (double)Wq[qi][dd];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const double df = (double)Wp[pi + 8 * t][dd] - b;
                s[t] = fma(df, df, s[t]);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int p = p0 + pi + 8 * t, q = q0 + qi;
        if (p < K && q < K) d2[(size_t)p * K + q] = s[t];
    }
}

// adjacency matrix A (K x K bytes) <- minimum spanning tree.  Ties between equal keys go to the lowest node index.  The
// rounds end early where no distance that is a number joins another node to the tree: those nodes stay apart.
__global__ void __launch_bounds__(1024) mst_prim_kernel(const double* __restrict__ d2, int K, unsigned char* __restrict__ A)
{
    extern __shared__ double prim_lds[];
    double* key = prim_lds;                                   // [K] cheapest connection to the tree
    int* from = reinterpret_cast<int*>(key + K);              // [K] its tree end
    __shared__ double red_v[16];
    __shared__ int red_i[16];
    __shared__ int chosen;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (size_t e = tid; e < (size_t)K * K; e += 1024) A[e] = 0;
    for (int v = tid; v < K; v += 1024) {
        key[v] = (v == 0) ? -1.0 : d2[v];                     // node 0 starts the tree; -1 marks "in tree"
        from[v] = 0;
    }
    __syncthreads();
    for (int round = 1; round < K; ++round) {
        double bv = INFINITY;
        int bi = 0x7fffffff;
        for (int v = tid; v < K; v += 1024) {
            const double k = key[v];
            if (k >= 0.0 && (k < bv || (k == bv && v < bi))) {
                bv = k;
                bi = v;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double ov = __shfl_xor(bv, o);
            const int oi = __shfl_xor(bi, o);
            if (ov < bv || (ov == bv && oi < bi)) {
                bv = ov;
                bi = oi;
            }
        }
        if (lane == 0) {
            red_v[wave] = bv;
            red_i[wave] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            double mv = red_v[0];
            int mi = red_i[0];
            for (int w = 1; w < 16; ++w)
                if (red_v[w] < mv || (red_v[w] == mv && red_i[w] < mi)) {
                    mv = red_v[w];
                    mi = red_i[w];
                }
            chosen = mi;
            if (mi < K) {
                const int f = from[mi];
                A[(size_t)mi * K + f] = 1;
                A[(size_t)f * K + mi] = 1;
                key[mi] = -1.0;
            }
        }
        __syncthreads();
        const int u = chosen;
        if (u >= K) break;
        const double* row = d2 + (size_t)u * K;
        for (int v = tid; v < K; v += 1024) {
            const double k = key[v];
            const double c = row[v];
            if (k >= 0.0 && c < k) {
                key[v] = c;
                from[v] = u;
            }
        }
        __syncthreads();
    }
}

// ---- Boruvka's method for K <= 4096: every round each component picks its cheapest outgoing edge under the strict
// order (length, lower end, higher end) -- the order Kruskal's method would visit edges in, so the tree is the
// same one even when lengths tie -- and the components joined by the picked edges merge.  At most ceil(log2 K)
// rounds; a round is one scan over all pairs (all compute units) and one single-workgroup merge.

__device__ __forceinline__ bool edge_before(double wa, int la, int ha, double wb, int lb, int hb)
{
    return wa < wb || (wa == wb && (la < lb || (la == lb && ha < hb)));
}

// state[0] = number of components, comp[v] = label of v's component (the label is one of its nodes)
__global__ void __launch_bounds__(256) boruvka_init_kernel(int K, int* __restrict__ comp, int* __restrict__ state,
                                                           unsigned char* __restrict__ A)
{
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e < (size_t)K * K) A[e] = 0;
    if (e < (size_t)K) comp[e] = (int)e;
    if (e == 0) state[0] = K;
}

// one wavefront per node v: cheapest edge to a node of another component, eight loads under way (each behind its component's test, a first
// round at K = 1024 took 13.5 us instead of 7.8)
__global__ void __launch_bounds__(256) boruvka_scan_kernel(const double* __restrict__ d2, int K, const int* __restrict__ comp,
                                                           const int* __restrict__ state, double* __restrict__ best_w,
                                                           int* __restrict__ best_u)
{
    if (state[0] <= 1) return;
    const int v = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (v >= K) return;
    const int cv = comp[v];
    double bw = INFINITY;
    int bu = -1;
    auto before = [&](double w, int u) {                       // (v, u) before the best so far
        return bu < 0 || edge_before(w, v < u ? v : u, v < u ? u : v, bw, v < bu ? v : bu, v < bu ? bu : v);
    };
    for (int u0 = lane; u0 < K; u0 += 8 * 64) {
        double w[8];
        int c[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int u = u0 + 64 * t < K ? u0 + 64 * t : u0;
            c[t] = comp[u];
            w[t] = d2[(size_t)v * K + u];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int u = u0 + 64 * t;
            if (u < K && c[t] != cv && before(w[t], u)) {
                bw = w[t];
                bu = u;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double ow = __shfl_xor(bw, o);
        const int ou = __shfl_xor(bu, o);
        if (ou >= 0 && before(ow, ou)) {
            bw = ow;
            bu = ou;
        }
    }
    if (lane == 0) {
        best_w[v] = bw;
        best_u[v] = bu;
    }
}

// single workgroup: per-component minimum of the node picks, edges into A, merge of the joined components.  A chain of latencies: what a
// thread needs of its nodes comes in at once and stays in registers, the labels in LDS, and pointers jump in place until none moves
// (three trips to memory, one more for the labels of an edge's ends, and log2 K jumps each time: whole call for data rows as nodes K = 4096
// 472 us, 407 this way, K = 1024 117 and 112).
constexpr int kMergeEach = kBoruvkaMaxNodes / 1024;
__global__ void __launch_bounds__(1024) boruvka_merge_kernel(int K, int* __restrict__ comp, int* __restrict__ state,
                                                             const double* __restrict__ best_w, const int* __restrict__ best_u,
                                                             unsigned char* __restrict__ A)
{
    if (state[0] <= 1) return;
    extern __shared__ unsigned long long bor_lds[];
    unsigned long long* cw = bor_lds;                                 // [K] bit pattern of the cheapest length
    unsigned long long* ce = cw + K;                                  // [K] its ends, lower << 32 | higher
    int* parent = reinterpret_cast<int*>(ce + K);                     // [K]
    int* label = parent + K;                                          // [K] comp
    __shared__ int count;
    const int tid = threadIdx.x;
    int mine[kMergeEach], other[kMergeEach];
    unsigned long long length[kMergeEach];
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int v = tid + 1024 * t;
        mine[t] = v < K ? comp[v] : 0;
        other[t] = v < K ? best_u[v] : -1;
        length[t] = v < K ? (unsigned long long)__double_as_longlong(best_w[v]) : 0ull;
    }
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int v = tid + 1024 * t;
        if (v < K) {
            cw[v] = ~0ull;
            ce[v] = ~0ull;
            label[v] = mine[t];
        }
    }
    if (tid == 0) count = 0;
    __syncthreads();
    // lengths are non-negative doubles (or +inf): their bit patterns order like the values
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t)
        if (other[t] >= 0) atomicMin(&cw[mine[t]], length[t]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int v = tid + 1024 * t, u = other[t];
        if (u >= 0 && length[t] == cw[mine[t]]) {
            const unsigned long long lo = v < u ? v : u, hi = v < u ? u : v;
            atomicMin(&ce[mine[t]], (lo << 32) | hi);
        }
    }
    __syncthreads();
    int par[kMergeEach];
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int c = tid + 1024 * t;
        par[t] = c;
        if (c < K && mine[t] == c && ce[c] != ~0ull) {
            const int lo = (int)(ce[c] >> 32), hi = (int)(ce[c] & 0xffffffffull);
            A[(size_t)lo * K + hi] = 1;
            A[(size_t)hi * K + lo] = 1;
            par[t] = label[lo] == c ? label[hi] : label[lo];
        }
        if (c < K) parent[c] = par[t];
    }
    __syncthreads();
    // two components that picked each other (necessarily the same edge): the lower label becomes the root
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int c = tid + 1024 * t;
        if (c < K && parent[par[t]] == c && c < par[t]) par[t] = c;
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t)
        if (tid + 1024 * t < K) parent[tid + 1024 * t] = par[t];
    __syncthreads();
    // (a pointer is one word and always leads to a node further on: no second copy; the rounds are bounded for weights that are no numbers)
    for (int span = 1; span < K; span <<= 1) {
        bool moved = false;
#pragma unroll
        for (int t = 0; t < kMergeEach; ++t) {
            const int c = tid + 1024 * t;
            if (c < K) {
                const int next = parent[par[t]];
                moved = moved || next != par[t];
                par[t] = next;
                parent[c] = next;
            }
        }
        if (!__syncthreads_or(moved)) break;
    }
    int roots = 0;
#pragma unroll
    for (int t = 0; t < kMergeEach; ++t) {
        const int v = tid + 1024 * t;
        if (v < K) {
            const int root = parent[mine[t]];
            comp[v] = root;
            if (root == v) ++roots;
        }
    }
    if (roots > 0) atomicAdd(&count, roots);
    __syncthreads();
    if (tid == 0) state[0] = count;
}

// Relative neighbourhood graph: pair (p, q) is an edge unless some third node r has
// max(d2[p][r], d2[q][r]) < d2[p][q].  Testing every r for every pair is K^3 / 2 comparisons, and almost every pair
// is blocked by a node close to one of its ends, so the test runs in three steps, all on the float64 distances:
//   rng_near_kernel       64 nodes near p for every p (the nearest one of every residue class modulo 64)
//   rng_prefilter_kernel  every pair against the 64 nodes near its lower end, nearest first; A = 1 where none blocks
//   rng_verify_kernel     the pairs left (the edges and a few more) against all nodes
// A blocker found in the second step is a blocker; a pair the second step leaves gets the complete test.  The
// result is the one the plain triple loop gives.
constexpr int kNear = 64;

__global__ void __launch_bounds__(256) rng_near_kernel(const double* __restrict__ d2, int K, int* __restrict__ near)
{
    const int lane = threadIdx.x & 63;
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (p >= K) return;
    const double* row = d2 + (size_t)p * K;
    double bv = INFINITY;
    int br = -1;
    for (int r = lane; r < K; r += kNear) {
        const double v = row[r];
        if (r != p && v < bv) {
            bv = v;
            br = r;
        }
    }
    near[(size_t)p * kNear + lane] = br;
}

// one workgroup per lower end p; thread -> upper ends q = tid, tid + 512, ...; eight of the near nodes' distances at a time, a trip to L2 each.
// K = 1024, the map of 4 * 10^7 x 50, 24 us (44 with one at a time and half as many threads), data rows as nodes 35 (66); K = 4096 197 (386)
constexpr int kPrefilterThreads = 512;
__global__ void __launch_bounds__(kPrefilterThreads) rng_prefilter_kernel(const double* __restrict__ d2, int K,
                                                            const int* __restrict__ near, unsigned char* __restrict__ A)
{
    __shared__ int nr_in[kNear], nr[kNear];
    __shared__ double dpr_in[kNear], dpr[kNear];
    const int tid = threadIdx.x, p = blockIdx.x;
    const double* rp = d2 + (size_t)p * K;
    if (tid < kNear) {
        const int r = near[(size_t)p * kNear + tid];
        nr_in[tid] = r;
        dpr_in[tid] = (r >= 0) ? rp[r] : INFINITY;
    }
    __syncthreads();
    if (tid < kNear) {
        // nearest first (rank by distance, then by place): the closest nodes block most pairs
        const double mine = dpr_in[tid];
        int rank = 0;
        for (int o = 0; o < kNear; ++o) rank += (dpr_in[o] < mine || (dpr_in[o] == mine && o < tid)) ? 1 : 0;
        nr[rank] = nr_in[tid];
        dpr[rank] = mine;
    }
    __syncthreads();
    for (int q = tid; q < K; q += kPrefilterThreads) {
        if (q == p) A[(size_t)p * K + p] = 0;
        if (q <= p) continue;
        const double lim = rp[q];
        bool blocked = false;
        for (int o = 0; o < kNear && !blocked; o += 8) {
            if (!(dpr[o] < lim)) break;                       // sorted: no later node is closer to p than the pair is long
            double v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = d2[(size_t)(nr[o + t] < 0 ? 0 : nr[o + t]) * K + q];
#pragma unroll
            for (int t = 0; t < 8; ++t) blocked = blocked || (dpr[o + t] < lim && v[t] < lim);
        }
        const unsigned char keep = blocked ? 0 : 1;
        A[(size_t)p * K + q] = keep;
        A[(size_t)q * K + p] = keep;
    }
}

// one workgroup per lower end p; a wavefront takes the surviving pairs of 64 upper ends at a time, all its lanes
// scan the third nodes of one pair together, 512 of them with their loads under way (256, and four wavefronts instead of
// eight: K = 1024 45 us, 12 this way; K = 4096 673 and 221)
constexpr int kVerifyThreads = 512;
__global__ void __launch_bounds__(kVerifyThreads) rng_verify_kernel(const double* __restrict__ d2, int K, unsigned char* __restrict__ A)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, p = blockIdx.x;
    const double* rp = d2 + (size_t)p * K;
    for (int qb = wave * 64; qb < K; qb += kVerifyThreads) {
        const int q = qb + lane;
        const bool alive = q > p && q < K && A[(size_t)p * K + q] != 0;
        unsigned long long mask = __ballot(alive);
        while (mask != 0ull) {
            const int qq = qb + (int)__ffsll((long long)mask) - 1;
            mask &= mask - 1ull;
            const double lim = rp[qq];
            const double* rq = d2 + (size_t)qq * K;
            bool found = false;
            // r = p and r = q give max = d2[p][q] itself, never strictly smaller: no masking needed
            for (int r0 = 0; r0 < K; r0 += 8 * 64) {
                double a[8], c[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int r = r0 + 64 * u + lane < K ? r0 + 64 * u + lane : K - 1;
                    a[u] = rp[r];
                    c[u] = rq[r];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) found = found || (fmax(a[u], c[u]) < lim);
                if (__any(found)) break;
            }
            if (__any(found) && lane == 0) {
                A[(size_t)p * K + qq] = 0;
                A[(size_t)qq * K + p] = 0;
            }
        }
    }
}

__global__ void __launch_bounds__(256) csr_degree_kernel(const unsigned char* __restrict__ A, int K, int* __restrict__ deg)
{
    const int v = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (v >= K) return;
    int c = 0;
    for (int u = lane; u < K; u += 64) c += A[(size_t)v * K + u] ? 1 : 0;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) deg[v] = c;
}

// off[0 .. K]: where the nodes' lists begin
__global__ void __launch_bounds__(1024) csr_scan_kernel(const int* __restrict__ deg, int K, int* __restrict__ off)
{
    __shared__ int part[1024];
    const int tid = threadIdx.x;
    const int per = (K + 1023) / 1024;
    int s = 0;
    for (int t = 0; t < per; ++t) {
        const int v = tid * per + t;
        if (v < K) s += deg[v];
    }
    part[tid] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int add = (tid >= o) ? part[tid - o] : 0;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    int run = part[tid] - s;
    for (int t = 0; t < per; ++t) {
        const int v = tid * per + t;
        if (v < K) {
            off[v] = run;
            run += deg[v];
        }
    }
    if (tid == 1023) off[K] = part[1023];
}

__global__ void __launch_bounds__(256) csr_fill_kernel(const unsigned char* __restrict__ A, int K,
                                                       const int* __restrict__ off, int* __restrict__ nbr)
{
    const int v = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (v >= K) return;
    int base = off[v];
    for (int u0 = 0; u0 < K; u0 += 64) {
        const int u = u0 + lane;
        const bool on = u < K && A[(size_t)v * K + u];
        const unsigned long long bal = __ballot(on);
        const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0));
        if (on) nbr[base + below] = u;
        base += __popcll(bal);
    }
}

constexpr size_t kTreeLds = 160 * 1024;

// Hop counts from a source to every node: one wavefront per source, no barriers.  A bit a node (visited) and the visiting
// order (uint16 queue, every node enters once) live in LDS; the frontier is the queue segment
// [head, tail).  Lanes take one frontier node each (or a share of it) and walk its neighbour list in step; a neighbour is claimed by
// setting its bit, and the claimed ones of a step are appended through a ballot (the queue
// position is a wave-uniform register, not a counter in memory).  LDS operations of one wavefront execute in
// order, so a later step sees the earlier steps' claims and queue entries.
__host__ __device__ constexpr size_t bfs_bits_bytes(int K) { return ((size_t)K + 31) / 32 * 4; }
__host__ __device__ constexpr size_t bfs_source_bytes(int K) { return bfs_bits_bytes(K) + ((size_t)K + 1) / 2 * 4; }       // LDS of a source

template <typename T>
__device__ __forceinline__ void bfs_source(const T* __restrict__ off, const T* __restrict__ nbr, int K, int src, unsigned int* seen,
                                           float* __restrict__ G)
{
    unsigned short* queue = reinterpret_cast<unsigned short*>(seen + bfs_bits_bytes(K) / 4);       // [K]
    float* const row = G + (size_t)src * K;
    const int lane = threadIdx.x & 63;
    for (int v = lane; v < (K + 31) / 32; v += 64) seen[v] = v == src >> 5 ? 1u << (src & 31) : 0u;
    if (lane == 0) {
        queue[0] = (unsigned short)src;
        row[src] = 0.0f;
    }
    int head = 0, tail = 1;
    for (int level = 0; head < tail; ++level) {
        const int end = tail;
        const int share = end - head <= 16 ? 2 : end - head <= 32 ? 1 : 0;      // a small level's nodes have four or two lanes each
        for (int base = head; base < end; base += 64 >> share) {
            const int i = base + (lane >> share);
            const bool has = i < end;
            const int v = has ? (int)queue[i] : 0;
            int e = has ? (int)off[v] + (lane & ((1 << share) - 1)) : 0;
            const int e1 = has ? (int)off[v + 1] : 0;
            while (__any(e < e1)) {
                bool won = false;
                int u = 0;
                if (e < e1) {
                    u = (int)nbr[e];
                    e += 1 << share;
                    won = (atomicOr(&seen[u >> 5], 1u << (u & 31)) >> (u & 31) & 1u) == 0u;
                }
                const unsigned long long mask = __ballot(won);
                if (won) {
                    const int below = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
                    queue[tail + below] = (unsigned short)u;
                    row[u] = (float)(level + 1);
                }
                tail += __popcll(mask);
            }
        }
        head = end;
    }
    if (tail < K)
        for (int v = lane; v < K; v += 64)
            if ((seen[v >> 5] >> (v & 31) & 1u) == 0u) row[v] = INFINITY;
}

// Up to sixteen sources a workgroup, which share the adjacency lists, as 16-bit numbers in LDS, where they fit what is left of it (`room` entries): a
// level is two dependent reads of the lists.  K = 1024, the map of 4 * 10^7 x 50, 38 us (54 with the lists in L2, a lane a node and the distances in
// LDS beside the queue); data rows as nodes 79 (84), K = 4096 1164 (1241).
constexpr int kBfsSources = 16;
__host__ __device__ constexpr size_t bfs_offset_bytes(int K) { return ((size_t)K + 2) / 2 * 4; }            // [K + 1] uint16

__global__ void __launch_bounds__(64 * kBfsSources) bfs_kernel(const int* __restrict__ off, const int* __restrict__ nbr, int K, int room,
                                                               float* __restrict__ G)
{
    extern __shared__ unsigned int bfs_lds[];
    const int waves = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), src = blockIdx.x * waves + wave;
    unsigned int* const own = bfs_lds + wave * (bfs_source_bytes(K) / 4);
    const int nnz = off[K];
    if (room == 0 || nnz > room) {                            // (the same for all)
        if (src < K) bfs_source(off, nbr, K, src, own, G);
        return;
    }
    unsigned short* const begin = reinterpret_cast<unsigned short*>(bfs_lds + waves * (bfs_source_bytes(K) / 4));
    unsigned short* const list = begin + bfs_offset_bytes(K) / 2;
    for (int v = threadIdx.x; v <= K; v += blockDim.x) begin[v] = (unsigned short)off[v];
    for (int e = threadIdx.x; e < nnz; e += blockDim.x) list[e] = (unsigned short)nbr[e];
    __syncthreads();
    if (src < K) bfs_source(begin, list, K, src, own, G);
}

// Hop counts of a spanning tree.  With the nodes in depth-first order, the last common ancestor of the nodes at places p < q lies one above the
// shallowest node of the places (p, q], or is the node at p itself; so a source's distances to all nodes are a running minimum of
// depths along the order, to either side of it.  (Walks along the branches, a lane each, took a step of LDS latency a level:
// 186 us for the trained map of 10^7 x 50 on 1024 nodes, 13 + 13 now; whole call for nodes along a line 347 and 136 us at K = 1024,
// 3982 and 646 at 4096, for data rows as nodes 169 and 117, 991 and 472.)
//
// The order: every edge once in each direction, one behind the other around the tree (the Euler tour: behind (u, v) comes v's edge after the
// one to u, in a circle), cut at node 0.  Places along the tour by pointer jumping (list ranking, Wyllie's), then depths by a sum over it.
// One workgroup, bound by the latency of log2(2 K) rounds.  An edge's word holds where it points (END: nowhere) and how many edges on that
// is; both change together and are true at any time, so a round needs no second copy.
// tour[place]: node, depth from bit 16.  state[1]: whether the graph is one tree of all nodes (weights that are no numbers can give another).
constexpr int kTourThreads = 1024;
// bytes of LDS: per directed edge (2 (K - 1)) its word, its end and its way back; per node where its edges begin; a word for votes
// (the sums of the wavefronts take the place of the edges' words in the end)
__host__ __device__ constexpr size_t tour_vote(int K) { return K < 16 ? 256 : ((size_t)K * 18 - 14 + 3) / 4 * 4; }
__host__ __device__ constexpr size_t tour_bytes(int K) { return tour_vote(K) + 4; }
constexpr int kTourNodes = (int)((kTreeLds - 4 + 14) / 18);       // most that fit (9102)
static_assert(tour_bytes(kTourNodes) <= kTreeLds && tour_bytes(kTourNodes + 1) > kTreeLds, "kTourNodes");
static_assert(2 * (kTourNodes - 1) < 0xffff && kTourNodes < 0x8000, "numbers of edges in sixteen bits, of nodes in fifteen");

__global__ void __launch_bounds__(kTourThreads) tree_tour_kernel(const int* __restrict__ off, const int* __restrict__ nbr, int K,
                                                                unsigned short* __restrict__ seq, unsigned int* __restrict__ tour,
                                                                int* __restrict__ state)
{
    extern __shared__ unsigned int tour_lds[];
    const int E = 2 * (K - 1), tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    unsigned int* const word = tour_lds;                                               // [E] next edge, edges up to there from bit 16
    unsigned short* const end = reinterpret_cast<unsigned short*>(word + E);           // [E]
    unsigned short* const back = end + E;                                              // [E]
    unsigned short* const begin = back + E;                                            // [K + 1]
    int2* const sums = reinterpret_cast<int2*>(tour_lds);                              // [wavefront]
    volatile int* const vote = reinterpret_cast<int*>(tour_lds + tour_vote(K) / 4);
    auto all = [&](bool yes) {
        if (tid == 0) *vote = 1;
        __syncthreads();
        if (!yes) *vote = 0;
        __syncthreads();
        const bool agreed = *vote != 0;
        __syncthreads();
        return agreed;
    };
    constexpr unsigned kEnd = 0xffffu;
    bool tree = off[K] == E;
    if (tree) {                                            // (the same for all)
        for (int v = tid; v <= K; v += kTourThreads) begin[v] = (unsigned short)off[v];
        for (int e = tid; e < E; e += kTourThreads) end[e] = (unsigned short)nbr[e];
    }
    __syncthreads();
    if (tree) {
        for (int v = tid; v < K; v += kTourThreads) tree = tree && (K == 1 || begin[v + 1] > begin[v]);
        for (int e = tid; e < E; e += kTourThreads) {
            int u = 0, top = K;                            // whose edge it is: the last node that begins at or before it
            while (top - u > 1) {
                const int mid = (u + top) >> 1;
                if ((int)begin[mid] <= e) u = mid;
                else top = mid;
            }
            const int v = end[e], first = begin[v], last = begin[v + 1];
            int t = first, above = last;                   // v's edge to u (lists are in ascending order)
            while (above - t > 1) {
                const int mid = (t + above) >> 1;
                if ((int)end[mid] <= u) t = mid;
                else above = mid;
            }
            back[e] = (unsigned short)t;
            const int next = t + 1 < last ? t + 1 : first;
            word[e] = (next == 0 ? kEnd : (unsigned)next) | 1u << 16;      // (node 0's first edge is edge 0)
        }
    }
    tree = all(tree);
    for (int reach = 1; tree && reach < E; reach <<= 1) {
        for (int e = tid; e < E; e += kTourThreads) {
            const unsigned w = word[e], n = w & 0xffffu;
            if (n != kEnd) {
                const unsigned x = word[n];
                word[e] = (x & 0xffffu) | ((w >> 16) + (x >> 16)) << 16;
            }
        }
        __syncthreads();
    }
    if (tree)
        for (int e = tid; e < E; e += kTourThreads) tree = tree && (word[e] & 0xffffu) == kEnd;
    tree = all(tree);
    if (tid == 0) state[1] = tree ? 1 : 0;
    if (!tree) return;
    // ends along the tour, and whether an edge leads away from node 0 (its way back comes later)
    for (int e = tid; e < E; e += kTourThreads) {
        const unsigned left = word[e] >> 16;
        seq[E - (int)left] = (unsigned short)(end[e] | (left > word[back[e]] >> 16 ? 0x8000u : 0u));
    }
    __syncthreads();
    // every thread takes a run of the tour: steps away less steps back, and steps away
    const int per = (E + kTourThreads - 1) / kTourThreads, lo = tid * per < E ? tid * per : E, hi = lo + per < E ? lo + per : E;
    int2 mine = make_int2(0, 0);
    for (int i = lo; i < hi; ++i) {
        const bool away = (seq[i] & 0x8000u) != 0u;
        mine.x += away ? 1 : -1;
        mine.y += away ? 1 : 0;
    }
    int2 at = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(at.x, o), y = __shfl_up(at.y, o);
        at.x += lane >= o ? x : 0;
        at.y += lane >= o ? y : 0;
    }
    if (lane == 63) sums[wave] = at;
    __syncthreads();
    int depth = at.x - mine.x, place = at.y - mine.y;
    for (int w = 0; w < wave; ++w) {
        depth += sums[w].x;
        place += sums[w].y;
    }
    if (tid == 0) tour[0] = 0u;
    for (int i = lo; i < hi; ++i) {
        const unsigned v = seq[i];
        depth += (v & 0x8000u) ? 1 : -1;
        if (v & 0x8000u) tour[++place] = (v & 0x7fffu) | (unsigned)depth << 16;
    }
}

// A wavefront a source, sixty-four places at a time; the row goes through LDS so that its lines are written whole.
constexpr int kTreeSources = 4;
__host__ __device__ constexpr size_t tree_source_bytes(int K) { return (size_t)K * 4 + 4; }      // (a row; a search takes less)

__global__ void __launch_bounds__(64 * kTreeSources) tree_hops_kernel(const int* __restrict__ off, const int* __restrict__ nbr, int K,
                                                                      const unsigned int* __restrict__ tour, const int* __restrict__ state,
                                                                      float* __restrict__ G)
{
    extern __shared__ unsigned int tree_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int src = blockIdx.x * (int)(blockDim.x >> 6) + wave;
    if (src >= K) return;                                     // (no barrier below)
    unsigned int* const own = tree_lds + wave * (tree_source_bytes(K) / 4);
    if (state[1] == 0) {
        bfs_source(off, nbr, K, src, own, G);
        return;
    }
    float* const row = reinterpret_cast<float*>(own);
    const unsigned here = tour[src];
    const int u = (int)(here & 0xffffu), du = (int)(here >> 16);
    if (lane == 0) row[u] = 0.0f;
    auto lowest = [&](int x) {                                // of this lane and those before it
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o);
            x = lane >= o && y < x ? y : x;
        }
        return x;
    };
    constexpr int kFar = 0x7fff;
    int low = du;                                             // depth of the common ancestor so far
    for (int q0 = src + 1; q0 < K; q0 += 64) {
        const int q = q0 + lane;
        const unsigned t = tour[q < K ? q : K - 1];
        const int d = (int)(t >> 16);
        int x = lowest(q < K ? d - 1 : kFar);
        x = x < low ? x : low;
        if (q < K) row[t & 0xffffu] = (float)(du + d - 2 * x);
        low = __shfl(x, 63);
    }
    low = du - 1;                                             // one above the shallowest of the places passed
    for (int q0 = src - 1; q0 >= 0; q0 -= 64) {
        const int q = q0 - lane;
        const unsigned t = tour[q >= 0 ? q : 0];
        const int d = (int)(t >> 16), x = lowest(q >= 0 ? d - 1 : kFar);
        int before = __shfl_up(x, 1);
        before = lane > 0 && before < low ? before : low;
        const int c = d < before ? d : before;
        if (q >= 0) row[t & 0xffffu] = (float)(du + d - 2 * c);
        const int all = __shfl(x, 63);
        low = all < low ? all : low;
    }
    __builtin_amdgcn_wave_barrier();
    for (int v = lane; v < K; v += 64) G[(size_t)u * K + v] = row[v];
}

} // namespace som

using namespace som;

extern "C" int som_topology(som_ctx* ctx, const float* W, int32_t K, int32_t D, int kind, float* G)
{
    if (!ctx) return SOM_EINVAL;
    if (!W || !G) return fail(ctx, SOM_EINVAL, "null W or G");
    if (K < 1 || D < 1) return fail(ctx, SOM_EINVAL, "K and D must be positive");
    if (kind != SOM_TOPOLOGY_MST && kind != SOM_TOPOLOGY_RNG) return fail(ctx, SOM_EINVAL, "unknown topology kind %d", kind);
    if (K > 12000) return fail(ctx, SOM_EINVAL, "K = %d is above the 12000 nodes the graph kernels hold in LDS", K);
    if (int rc = check_hip(ctx, hipSetDevice(ctx->device), "hipSetDevice")) return rc;
    const size_t kk = (size_t)K * K;
    const size_t need = kk * sizeof(double) + (size_t)K * sizeof(double) + ((size_t)4 * K + 8 + kk) * sizeof(int) + kk + 1024 +
                        (size_t)K * kNear * sizeof(int);
    if (need > ctx->topo_bytes) {
        if (ctx->topo_blob) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->topo_blob);
            ctx->topo_blob = nullptr;
            ctx->topo_bytes = 0;
        }
        if (hipMalloc(&ctx->topo_blob, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the topology workspace", need);
        }
        ctx->topo_bytes = need;
    }
    double* d2 = (double*)ctx->topo_blob;
    double* best_w = d2 + kk;
    int* deg = (int*)(best_w + K);
    int* off = deg + K;                                  // K + 1 entries
    int* comp = off + K + 1;
    int* best_u = comp + K;
    int* state = best_u + K;                             // 4 entries
    int* nbr = state + 4;                                // at most K * K entries
    unsigned char* A = (unsigned char*)(nbr + kk);
    int* near = (int*)(A + (kk + 1023) / 1024 * 1024);   // K * kNear entries (relative neighbourhood graph only)
    const dim3 tiles((K + 31) / 32, (K + 31) / 32);
    hipLaunchKernelGGL(node_d2_kernel, tiles, dim3(256), 0, ctx->stream, W, K, D, d2);
    if (int rc = check_hip(ctx, hipGetLastError(), "node distance launch")) return rc;
    if (kind == SOM_TOPOLOGY_MST && K <= kBoruvkaMaxNodes) {
        const size_t lds = (size_t)K * 24;
        if (lds > 48 * 1024) {
            if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(boruvka_merge_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kBoruvkaMaxNodes * 24), "raising the dynamic LDS limit")) return rc;
        }
        hipLaunchKernelGGL(boruvka_init_kernel, dim3((unsigned)((kk + 255) / 256)), dim3(256), 0, ctx->stream, K, comp, state, A);
        int rounds = 0;
        while ((1 << rounds) < K) ++rounds;              // the number of components at least halves every round
        for (int r = 0; r < rounds; ++r) {
            hipLaunchKernelGGL(boruvka_scan_kernel, dim3((K + 3) / 4), dim3(256), 0, ctx->stream, d2, K, comp, state, best_w, best_u);
            hipLaunchKernelGGL(boruvka_merge_kernel, dim3(1), dim3(1024), lds, ctx->stream, K, comp, state, best_w, best_u, A);
        }
    } else if (kind == SOM_TOPOLOGY_MST) {
        const size_t lds = (size_t)K * 12 + 16;
        if (lds > 48 * 1024) {
            if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(mst_prim_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024), "raising the dynamic LDS limit")) return rc;
        }
        hipLaunchKernelGGL(mst_prim_kernel, dim3(1), dim3(1024), lds, ctx->stream, d2, K, A);
    } else {
        hipLaunchKernelGGL(rng_near_kernel, dim3((K + 3) / 4), dim3(256), 0, ctx->stream, d2, K, near);
        hipLaunchKernelGGL(rng_prefilter_kernel, dim3(K), dim3(kPrefilterThreads), 0, ctx->stream, d2, K, near, A);
        hipLaunchKernelGGL(rng_verify_kernel, dim3(K), dim3(kVerifyThreads), 0, ctx->stream, d2, K, A);
    }
    if (int rc = check_hip(ctx, hipGetLastError(), "edge kernel launch")) return rc;
    hipLaunchKernelGGL(csr_degree_kernel, dim3((K + 3) / 4), dim3(256), 0, ctx->stream, A, K, deg);
    hipLaunchKernelGGL(csr_scan_kernel, dim3(1), dim3(1024), 0, ctx->stream, deg, K, off);
    hipLaunchKernelGGL(csr_fill_kernel, dim3((K + 3) / 4), dim3(256), 0, ctx->stream, A, K, off, nbr);
    if (int rc = check_hip(ctx, hipGetLastError(), "adjacency launch")) return rc;
    if (kind == SOM_TOPOLOGY_MST && K <= kTourNodes) {
        const size_t tour_lds = tour_bytes(K);
        int sources = kTreeSources;                      // of a workgroup
        while (sources * tree_source_bytes(K) > kTreeLds) --sources;
        const size_t lds = sources * tree_source_bytes(K);
        if (tour_lds > 48 * 1024) {
            if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(tree_tour_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTreeLds), "raising the dynamic LDS limit")) return rc;
        }
        if (lds > 48 * 1024) {
            if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(tree_hops_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTreeLds), "raising the dynamic LDS limit")) return rc;
        }
        // (best_u and comp have no more use: the order, and in front of it what the tour passes, 2 (K - 1) 16-bit words)
        hipLaunchKernelGGL(tree_tour_kernel, dim3(1), dim3(kTourThreads), tour_lds, ctx->stream, off, nbr, K, (unsigned short*)comp, (unsigned int*)best_u, state);
        if (int rc = check_hip(ctx, hipGetLastError(), "tree order launch")) return rc;
        hipLaunchKernelGGL(tree_hops_kernel, dim3((K + sources - 1) / sources), dim3(64 * sources), lds, ctx->stream, off, nbr, K, (const unsigned int*)best_u, state, G);
        return check_hip(ctx, hipGetLastError(), "hop-count launch");
    }
    // As many sources as give every compute unit one workgroup, and no more than leave room for six neighbours a node on average; the lists get
    // what LDS has left, up to sixteen a node.  Where they leave room for less than half of the sources that fit without them they stay in L2:
    // on 6000 nodes (8 features, six neighbours) 868 us with six sources and lists, 922 with twelve and none; on 7000 (four, eleven) 1682 and 1493,
    // 9000 (one, eight) 13,150 and 2830, 12,000 (one, six) 29,600 and 5730.  (A source a workgroup, its distances beside the queue: 1403, 2666, 6160,
    // 11,020.)
    const int even = (K + ctx->units - 1) / ctx->units, asked = even < 4 ? 4 : even > kBfsSources ? kBfsSources : even;
    auto sources_beside = [&](size_t lists) {
        int n = asked;
        while (n > 1 && n * bfs_source_bytes(K) + lists > kTreeLds) --n;
        return n;
    };
    const int beside = sources_beside(bfs_offset_bytes(K) + (size_t)K * 12), alone = sources_beside(0);
    const bool lists = 2 * beside + 1 >= alone;
    const int waves = lists ? beside : alone;
    const size_t own = waves * bfs_source_bytes(K) + (lists ? bfs_offset_bytes(K) : 0);
    size_t room = lists ? (kTreeLds - own) / 2 : 0;
    room = room < (size_t)K * 16 + 2 ? room : (size_t)K * 16 + 2;
    room = (room < 65535 ? room : 65535) / 2 * 2;
    const size_t bfs_lds_bytes = own + 2 * room;
    if (bfs_lds_bytes > 48 * 1024) {
        if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(bfs_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTreeLds), "raising the dynamic LDS limit")) return rc;
    }
    hipLaunchKernelGGL(bfs_kernel, dim3((K + waves - 1) / waves), dim3(64 * waves), bfs_lds_bytes, ctx->stream, off, nbr, K, (int)room, G);
    return check_hip(ctx, hipGetLastError(), "hop-count launch");
}
