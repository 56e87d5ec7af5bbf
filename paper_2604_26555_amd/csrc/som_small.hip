// Small calls: maps and tables for which the search, the accumulation and the update are each a few microseconds of
// arithmetic, so that what counts is how many kernels there are.  The general path takes ten (centre, preparation,
// search, list, candidates, differences, sums, reduction, contraction, finish) of 2 to 25 us each; here a look-up is
// one kernel and an epoch two.
//
// Distances are the float32 direct differences sum_d (x_d - w_kd)^2, features in order, that the general path's
// re-decisions use (lowest distance, then lowest node index); so no bound, no list and no second decision.  The sums
// are float64, like the general path's.
//
//   small_kernel      a few lanes per sample (each takes every SUB-th node, W in LDS), rows of at most 32 features;
//                     with ACC the workgroup also adds its samples up in LDS and its sums onto the map's
//   lookup_kernel     a thread per node and 4 or 8 samples per workgroup (rows of at most 64 features, any map): W comes
//                     through LDS in pieces, the samples' values in scalar registers
//   small_update_kernel   four wavefronts per node: influences, the contraction over the nodes and the rule
#include "som_bmu_common.hpp"

#include <math.h>

namespace som {

constexpr int kSThreads = 512;
constexpr size_t kSLds = 128 * 1024;          // W and the sums of small_kernel, a piece of W in lookup_kernel
constexpr size_t kSCells = kSLds / sizeof(double);   // cells of a set of sums: they are in LDS beside W, so never as many
constexpr int kSFeatures = 32;                // small_kernel: features of a row at most
constexpr int kSNodes = 512;                  // small epochs: nodes at most
constexpr double kSWork = 3.0e8;              // m K D of a small epoch at most: 0.4 to 0.8 of the general path's time there (D = 2 ... 32,
                                              // K = 16 ... 512), at 6e8 0.5 to 1.3
// Small epochs: copies of the sums, one to an XCD's workgroups (they are dealt out in turn), where the eight fit into a set.
// Few cells are the ones that many workgroups meet in: 256 workgroups that added to one copy of 900 cells took 4000 to 6000 of
// small_kernel's 17,000 cycles for it.
constexpr int kSCopies = 8;
constexpr int kSFlight = 8;                   // lookup_kernel: loads of W under way in a thread
constexpr double kLWork = 4.0e8;              // ... of a small look-up,
constexpr double kLSteps = 6.0e8;             // and the same with rows and features rounded up (look_up_rows)

struct SmallArgs {
    const float* X;
    int64_t ldx;
    const uint32_t* idx;
    int64_t m;
    int D, K, sub;                            // sub: lanes per sample (a power of two)
    const float* W;
    int32_t* bmu;                             // may be null (epochs)
    float* d2;
    double* qe_part;                          // may be null
    double* S;                                // ACC: `copies` of [K][D + 1], the last column counts
    int copies;
};

// Where node k's row (dq float4) starts in LDS, in float4.  The lanes of a sample read neighbouring nodes' rows at once: rows
// of four or eight float4 are moved on by one float4 after every 256 bytes, or all of them start in the same few banks
// (32 features, 400 nodes, 1000 samples: 28.9 us without, 14 with; the general path takes 23).  Rows of two or six meet in
// pairs at most and stay as they are.
__host__ __device__ constexpr int small_row(int k, int dq) { return k * dq + (dq == 4 ? k >> 2 : dq == 8 ? k >> 1 : 0); }

// v of the lane that a DPP control names, ~0 where there is none
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ unsigned dpp(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(-1, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ unsigned less(unsigned a, unsigned b) { return a < b ? a : b; }
// the least of a full wavefront, for every lane
__device__ __forceinline__ unsigned wave_min(unsigned v)
{
    v = less(v, dpp<0x111>(v));              // one to the right in a row of sixteen,
    v = less(v, dpp<0x112>(v));              // two,
    v = less(v, dpp<0x114>(v));              // four,
    v = less(v, dpp<0x118>(v));              // eight: the row's last lane has its least
    v = less(v, dpp<0x142, 0xa>(v));         // which the next row takes over,
    v = less(v, dpp<0x143, 0xc>(v));         // and the upper half
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
// the least of each 2, 4, 8 or 16 lanes, for each of them
__device__ __forceinline__ unsigned min_of(unsigned v, int lanes)
{
    if (lanes > 1) v = less(v, dpp<0xb1>(v));        // neighbours,
    if (lanes > 2) v = less(v, dpp<0x4e>(v));        // pairs,
    if (lanes > 4) v = less(v, dpp<0x141>(v));       // halves of a row, mirrored,
    if (lanes > 8) v = less(v, dpp<0x140>(v));       // rows, mirrored
    return v;
}

// DQ: float4 of a row.  The first row of a thread is on its way while W is brought in, and a sample's lanes find its winner by
// DPP moves: with the copies of the sums, 10,000 rows of 8 features on 100 nodes 8.5 -> 5.7 us.
template <int DQ, bool ACC>
__global__ void __launch_bounds__(kSThreads) small_kernel(const SmallArgs a)
{
    extern __shared__ float4 small_lds[];
    float4* const w4 = small_lds;                                             // K rows of DQ, zeros behind the row
    double* const sums = reinterpret_cast<double*>(small_lds + small_row(a.K, DQ) + 1);   // ACC: [K][D + 1]
    const int tid = threadIdx.x, D = a.D, K = a.K, DS = D + 1;
    float* const wf = reinterpret_cast<float*>(w4);
    const int sub = tid & (a.sub - 1), per = kSThreads / a.sub;
    int64_t p0 = (int64_t)blockIdx.x * per;
    float x[4 * DQ];
    auto row = [&] {
        const int64_t i = p0 + tid / a.sub, ic = i < a.m ? i : a.m - 1;
        const float* xr = a.X + (a.idx ? (int64_t)a.idx[ic] : ic) * a.ldx;
#pragma unroll
        for (int q = 0; q < DQ; ++q) {
            if (4 * q + 4 <= D) {
                const float4 v = load4(xr + 4 * q);
                x[4 * q] = v.x;
                x[4 * q + 1] = v.y;
                x[4 * q + 2] = v.z;
                x[4 * q + 3] = v.w;
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) x[4 * q + t] = 4 * q + t < D ? xr[4 * q + t] : 0.0f;
            }
        }
    };
    row();                                                     // (on its way while W comes)
    for (int e = tid; e < K * DQ * 4; e += kSThreads) {
        const int k = e / (DQ * 4), f = e - k * (DQ * 4);
        wf[small_row(k, DQ) * 4 + f] = f < D ? a.W[(size_t)k * D + f] : 0.0f;
    }
    if constexpr (ACC)
        for (int e = tid; e < K * DS; e += kSThreads) sums[e] = 0.0;
    __syncthreads();
    double qs = 0.0, qs2 = 0.0;
    while (p0 < a.m) {
        const int64_t i = p0 + tid / a.sub;
        const bool live = i < a.m;
        float bd = INFINITY;
        int bk = 0x7fffffff;
        // two nodes at a time: two chains of additions
        for (int k = sub; k < K; k += 2 * a.sub) {
            const int k1 = k + a.sub < K ? k + a.sub : k;
            const float4 *r0 = w4 + small_row(k, DQ), *r1 = w4 + small_row(k1, DQ);
            float d0 = 0.0f, d1 = 0.0f;
#pragma unroll
            for (int q = 0; q < DQ; ++q) {
                const float4 u = r0[q], v = r1[q];
                const float wu[4] = {u.x, u.y, u.z, u.w}, wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float e0 = x[4 * q + t] - wu[t], e1 = x[4 * q + t] - wv[t];
                    d0 = fmaf(e0, e0, d0);
                    d1 = fmaf(e1, e1, d1);
                }
            }
            if (d0 < bd) {
                bd = d0;
                bk = k;
            }
            if (d1 < bd) {
                bd = d1;
                bk = k1;
            }
        }
        const unsigned bits = min_of(__float_as_uint(bd), a.sub);             // (no distance is negative or NaN)
        bk = (int)min_of(__float_as_uint(bd) == bits ? (unsigned)bk : 0x7fffffffu, a.sub);
        bd = __uint_as_float(bits);
        if (bk >= K) bk = 0;                                   // only reachable with non-finite input
        if (live && sub == 0) {
            if (a.bmu) a.bmu[i] = bk;
            if (a.d2) a.d2[i] = bd;
            qs += sqrt((double)bd);
            qs2 += (double)bd;
        }
        if constexpr (ACC) {
            // a sample's lanes share its features; the last place counts
            if (live) {
                double* s = sums + bk * DS;
#pragma unroll
                for (int f = 0; f < 4 * DQ; ++f)
                    if (f < D && (f & (a.sub - 1)) == sub) unsafeAtomicAdd(&s[f], (double)x[f]);
                if (sub == 0) unsafeAtomicAdd(&s[D], 1.0);
            }
        }
        p0 += (int64_t)gridDim.x * per;
        if (p0 < a.m) row();
    }
    if constexpr (ACC) {
        __syncthreads();
        double* const own = a.S + (size_t)(blockIdx.x % a.copies) * (K * DS);
        for (int e = tid; e < K * DS; e += kSThreads) {
            const double v = sums[e];
            if (v != 0.0) unsafeAtomicAdd(&own[e], v);
        }
    }
    if (a.qe_part) group_qe_add(a.qe_part, qs, qs2);
}

__device__ __forceinline__ double lane_value(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane), __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// S samples per workgroup; nodes in pieces of `piece` (their rows in LDS, `stride` floats apart, odd or harmless to the banks).
// A look-up is one round of workgroups, so what counts is the chain of waits in one of them.  Of the 27,500 cycles that a
// workgroup took for 4 samples of 50 features on 1024 nodes, 8000 brought W in (a load at a time in each thread: now kSFlight
// of them), 8100 were differences (6400 is what the vector units need) and 9600 the join of the threads' winners, where every
// step waited for a shuffle through LDS; DPP moves and one barrier do it in about 1500.  Look-ups with distances and
// quantisation error, in us: 1000 rows 15.4 -> 12.5, 12,288 rows of 50 features on 64 nodes 40.3 -> 32.1, 2000 of 37 on 400
// 15.5 -> 11.2, 4095 of 40 on 1500 43.3 -> 36.7, 300 of 64 on 20,000 248 -> 191.  The samples' rows in LDS in place of scalar
// loads: 13.1 against 12.4 (the broadcast reads cost more than the loads' latency).  Parts of the nodes on workgroups of their
// own, joined by the last to arrive: 15.7 against 15.4 at 1000 rows (faster only for a few rows on many nodes).
template <int S>
__global__ void __launch_bounds__(kSThreads) lookup_kernel(const float* __restrict__ X, const float* __restrict__ W, const SmallArgs a,
                                                           int piece, int stride)
{
    extern __shared__ float4 small_lds[];
    __shared__ uint2 red[S][kSThreads / 64];
    float* const wl = reinterpret_cast<float*>(small_lds);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, D = a.D, K = a.K;
    const int64_t i0 = (int64_t)blockIdx.x * S;
    // the samples' rows: the same for the whole workgroup, so that their values are scalar loads
    const float* xrow[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int64_t i = i0 + s < a.m ? i0 + s : a.m - 1;
        xrow[s] = X + (a.idx ? (int64_t)a.idx[i] : i) * a.ldx;
    }
    float bd[S];
    int bk[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        bd[s] = INFINITY;
        bk[s] = 0x7fffffff;
    }
    for (int k0 = 0; k0 < K; k0 += piece) {
        const int kn = K - k0 < piece ? K - k0 : piece;
        __syncthreads();
        // the piece's rows are contiguous in W
        const float* from = W + (size_t)k0 * D;
        if (stride == D) {
            const int words = kn * D, whole = words / 4;
            float4* to = reinterpret_cast<float4*>(wl);
#pragma nounroll
            for (int e = tid; e < whole; e += kSFlight * kSThreads) {
                float4 v[kSFlight];
#pragma unroll
                for (int t = 0; t < kSFlight; ++t) v[t] = load4(from + 4 * (e + t * kSThreads < whole ? e + t * kSThreads : e));
#pragma unroll
                for (int t = 0; t < kSFlight; ++t)
                    if (e + t * kSThreads < whole) to[e + t * kSThreads] = v[t];
            }
            for (int e = 4 * whole + tid; e < words; e += kSThreads) wl[e] = from[e];
        } else {
            const int dq = D / 4;                           // (a multiple of four: padded rows)
            const int whole = kn * dq;
#pragma nounroll
            for (int e = tid; e < whole; e += kSFlight * kSThreads) {
                float4 v[kSFlight];
#pragma unroll
                for (int t = 0; t < kSFlight; ++t) v[t] = load4(from + 4 * (e + t * kSThreads < whole ? e + t * kSThreads : e));
#pragma unroll
                for (int t = 0; t < kSFlight; ++t)
                    if (e + t * kSThreads < whole) {
                        const int r = (e + t * kSThreads) / dq, q = e + t * kSThreads - r * dq;
                        float* to = wl + r * stride + 4 * q;
                        to[0] = v[t].x;
                        to[1] = v[t].y;
                        to[2] = v[t].z;
                        to[3] = v[t].w;
                    }
            }
        }
        __syncthreads();
        for (int n = tid; n < kn; n += kSThreads) {
            const float* w = wl + n * stride;
            float d[S];
#pragma unroll
            for (int s = 0; s < S; ++s) d[s] = 0.0f;
            int f = 0;
            for (; f + 8 <= D; f += 8) {
                float wv[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) wv[t] = w[f + t];
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int s = 0; s < S; ++s) {
                        const float e = xrow[s][f + t] - wv[t];
                        d[s] = fmaf(e, e, d[s]);
                    }
            }
            for (; f < D; ++f) {
                const float wv = w[f];
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    const float e = xrow[s][f] - wv;
                    d[s] = fmaf(e, e, d[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < S; ++s)
                if (d[s] < bd[s]) {
                    bd[s] = d[s];
                    bk[s] = k0 + n;
                }
        }
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const unsigned d = wave_min(__float_as_uint(bd[s]));                  // (no distance is negative or NaN)
        const unsigned k = wave_min(__float_as_uint(bd[s]) == d ? (unsigned)bk[s] : 0x7fffffffu);
        if (lane == 0) red[s][wave] = make_uint2(d, k);
    }
    __syncthreads();
    if (wave != 0) return;
    // eight lanes to a sample
    static_assert(kSThreads == 8 * 64 && S <= 8, "a wavefront joins all samples' eight winners");
    const int s = lane >> 3;
    const uint2 mine = red[s < S ? s : 0][lane & 7];
    const unsigned bits = min_of(mine.x, 8);
    int k = (int)min_of(mine.x == bits ? mine.y : 0x7fffffffu, 8);
    const float d = __uint_as_float(bits);
    double qs = 0.0, qs2 = 0.0;
    if ((lane & 7) == 0 && s < S && i0 + s < a.m) {
        if (k >= K) k = 0;                                     // only reachable with non-finite input
        a.bmu[i0 + s] = k;
        if (a.d2) a.d2[i0 + s] = d;
        qs = sqrt((double)d);
        qs2 = (double)d;
    }
    if (a.qe_part) {
        double t0 = 0.0, t1 = 0.0;
#pragma unroll
        for (int t = 0; t < S; ++t) {
            t0 += lane_value(qs, 8 * t);
            t1 += lane_value(qs2, 8 * t);
        }
        if (lane == 0 && (t0 != 0.0 || t1 != 0.0)) {
            const int slot = blockIdx.x & (kQeSlots - 1);
            unsafeAtomicAdd(&a.qe_part[2 * slot], t0);
            unsafeAtomicAdd(&a.qe_part[2 * slot + 1], t1);
        }
    }
}

// qe[0..1] = the call's partial sums, which are left zero for the next call
__global__ void __launch_bounds__(kQeSlots) small_qe_kernel(double* __restrict__ part, double* __restrict__ qe)
{
    __shared__ double w[kQeSlots / 64][2];
    const int tid = threadIdx.x;
    double s0 = part[2 * tid], s1 = part[2 * tid + 1];
    part[2 * tid] = 0.0;
    part[2 * tid + 1] = 0.0;
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if ((tid & 63) == 0) {
        w[tid >> 6][0] = s0;
        w[tid >> 6][1] = s1;
    }
    __syncthreads();
    if (tid == 0) {
        double t0 = 0.0, t1 = 0.0;
        for (int q = 0; q < kQeSlots / 64; ++q) {
            t0 += w[q][0];
            t1 += w[q][1];
        }
        qe[0] = t0;
        qe[1] = t1;
    }
}

// The update of a small map (definitions in som_update.hip): kUNodes nodes j to a workgroup, kUWaves wavefronts to a node.
// S: `copies` (one or kSCopies) of [K][D + 1] float64 with the counts in the last column.  `clear`: the other call's sums, zero
// when the next call adds to them (null under capture).
// What counts is the chain of waits: distances and sums come in together, the sums through LDS (a wavefront that read them from
// memory for its node alone waited for every eight rows of its part), and a node's rows are shared by four wavefronts.  400
// nodes of 8 features 9.8 -> 5.2 us, 300 of 17 11.8 -> 6.0, 100 of 8 4.7 -> 4.5 with eight copies to add up instead of one.
constexpr int kUThreads = 512, kUNodes = 2, kUWaves = kUThreads / 64 / kUNodes;

__global__ void __launch_bounds__(kUThreads) small_update_kernel(const float* __restrict__ G, const double* __restrict__ S, int copies, int K,
                                                                 int D, double inv2s2, bool shifted, double eps_h, bool plain, double eta,
                                                                 double mu, float* __restrict__ V, float* __restrict__ W,
                                                                 double* __restrict__ clear)
{
    extern __shared__ float4 small_lds[];
    double* const sums = reinterpret_cast<double*>(small_lds);                // [K][D + 1]
    __shared__ double h_lds[kUNodes][kSNodes];
    __shared__ double join[kUNodes][kUWaves][64];
    constexpr int kPer = kUThreads / kUNodes;                                 // threads to a node
    const int tid = threadIdx.x, lane = tid & 63, node = tid / kPer, at = tid - node * kPer, wave = at >> 6, DS = D + 1, cells = K * DS;
    const int j = blockIdx.x * kUNodes + node, column = j < K ? j : K - 1;
    double g[(kSNodes + kPer - 1) / kPer];
#pragma unroll
    for (int t = 0; t < (kSNodes + kPer - 1) / kPer; ++t) {
        const int k = at + t * kPer;
        g[t] = (double)G[(size_t)(k < K ? k : K - 1) * K + column];
    }
    // all copies of two cells, or eight cells of the only copy, under way together
    if (copies == kSCopies) {
#pragma nounroll
        for (int e = tid; e < cells; e += 2 * kUThreads) {
            const int f = e + kUThreads < cells ? e + kUThreads : e;
            double v = 0.0, u = 0.0;
#pragma unroll
            for (int c = 0; c < kSCopies; ++c) {
                v += S[c * cells + e];
                u += S[c * cells + f];
            }
            sums[e] = v;
            sums[f] = f == e ? v : u;
        }
    } else {
#pragma nounroll
        for (int e = tid; e < cells; e += 8 * kUThreads) {
            double v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = S[e + t * kUThreads < cells ? e + t * kUThreads : e];
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (e + t * kUThreads < cells) sums[e + t * kUThreads] = v[t];
        }
    }
    if (clear)
        for (int e = blockIdx.x * kUThreads + tid; e < copies * cells; e += gridDim.x * kUThreads) clear[e] = 0.0;
    __syncthreads();
    double shift = 0.0;
    if (shifted) {
        shift = INFINITY;
#pragma unroll
        for (int t = 0; t < (kSNodes + kPer - 1) / kPer; ++t) {
            const int k = at + t * kPer;
            if (k < K && sums[k * DS + D] != 0.0 && g[t] * g[t] < shift) shift = g[t] * g[t];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) shift = fmin(shift, __shfl_xor(shift, o));
        if (lane == 0) join[node][wave][0] = shift;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kUWaves; ++w) shift = fmin(shift, join[node][w][0]);
    }
#pragma unroll
    for (int t = 0; t < (kSNodes + kPer - 1) / kPer; ++t) {
        const int k = at + t * kPer;
        const double e = -(g[t] * g[t] - shift) * inv2s2;
        const bool out = isinf(g[t]) || isinf(shift) || (shifted && sums[(k < K ? k : 0) * DS + D] == 0.0);
        if (k < K) h_lds[node][k] = out ? 0.0 : exp(e);
    }
    __syncthreads();
    // lanes: a column each, in 64 / width parts over a wavefront's share of the nodes
    int width = 1;
    while (width < DS) width <<= 1;
    const int c = lane & (width - 1), parts = 64 / width * kUWaves, part = wave * (64 / width) + lane / width;
    double num = 0.0;
    if (c < DS) {
#pragma unroll 4
        for (int k = part; k < K; k += parts) num += h_lds[node][k] * sums[k * DS + c];
    }
    for (int o = width; o < 64; o <<= 1) num += __shfl_xor(num, o);
    join[node][wave][lane] = num;
    __syncthreads();
    if (wave != 0 || lane >= D || j >= K) return;
    double den = 0.0;
    num = 0.0;
#pragma unroll
    for (int w = 0; w < kUWaves; ++w) {
        num += join[node][w][lane];
        den += join[node][w][D];
    }
    const size_t e = (size_t)j * D + lane;
    const bool ok = den >= eps_h;
    if (plain) {
        if (ok) W[e] = (float)(num / den);
    } else {
        const double w = (double)W[e];
        const double delta = (ok ? eta * (num / den - w) : 0.0) + (V ? mu * (double)V[e] : 0.0);
        W[e] = (float)(w + delta);
        if (V) V[e] = (float)delta;
    }
}

// ---------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------
// rows and sums of small_kernel; what the rows' places take beyond them (at most a sixteenth) is not counted here
static size_t small_lds_bytes(int K, int D, bool acc)
{
    return (size_t)K * ((D + 3) / 4) * 16 + (acc ? (size_t)K * (D + 1) * 8 : 0);
}

template <bool ACC>
static int launch_small(som_ctx* ctx, SmallArgs a, int blocks_most)
{
    // lanes per sample: enough threads for two wavefronts per SIMD, as long as every lane has nodes to look at
    a.sub = 1;
    while (a.sub < 16 && a.m * a.sub < 256 * 512 && a.sub * 8 <= a.K) a.sub <<= 1;
    const int64_t per = kSThreads / a.sub, need = (a.m + per - 1) / per;
    const unsigned blocks = (unsigned)(need < blocks_most ? need : blocks_most);
    const size_t lds = (size_t)(small_row(a.K, (a.D + 3) / 4) + 1) * 16 + (ACC ? (size_t)a.K * (a.D + 1) * 8 : 0);
    static bool attr_set_dev[kMaxDevices][9] = {};       // the attribute belongs to the device, not to the process
    const int dq = (a.D + 3) / 4;
    auto launch = [&](auto kern) -> int {
        bool& attr_set = attr_set_dev[ctx->device][dq];
        if (!attr_set) {
            if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kSLds + kSLds / 16)),
                                   "raising the dynamic LDS limit"))
                return rc;
            attr_set = true;
        }
        hipLaunchKernelGGL(kern, dim3(blocks), dim3(kSThreads), lds, ctx->stream, a);
        return check_hip(ctx, hipGetLastError(), "small-map kernel launch");
    };
    switch (dq) {
    case 1: return launch(small_kernel<1, ACC>);
    case 2: return launch(small_kernel<2, ACC>);
    case 3: return launch(small_kernel<3, ACC>);
    case 4: return launch(small_kernel<4, ACC>);
    case 5: return launch(small_kernel<5, ACC>);
    case 6: return launch(small_kernel<6, ACC>);
    case 7: return launch(small_kernel<7, ACC>);
    case 8: return launch(small_kernel<8, ACC>);
    }
    return fail(ctx, SOM_EINVAL, "no small-map kernel for %d features", a.D);
}

// LDS layout of lookup_kernel: rows of `stride` floats (one that is no multiple of four spreads a wavefront's reads over the
// banks), `piece` nodes at a time
struct LookupLds {
    int stride, piece;
    size_t bytes;
};
static LookupLds lookup_lds(int K, int D)
{
    LookupLds l;
    l.stride = D % 4 == 0 ? D + 1 : D;
    l.piece = (int)(kSLds / sizeof(float)) / l.stride;
    if (l.piece > kSThreads) l.piece = l.piece / kSThreads * kSThreads;
    if (l.piece > K) l.piece = K;
    l.bytes = ((size_t)l.piece * l.stride * sizeof(float) + 15) / 16 * 16;
    return l;
}

static bool lookup_in_lds(int K, int D) { return D <= kSFeatures && small_lds_bytes(K, D, false) <= kSLds / 2; }

// The most rows of a look-up that go through one kernel here; the others take the general path.  Both sides were timed over
// D = 3 ... 64, K = 16 ... 20000 and rows from 300 across the line, with and without distances, on rows that the caches hold
// and on rows that they do not.
// (Timed before the threads' winners were joined by DPP moves: a look-up takes 0.75 to 0.95 of those times now, so the lines
// are on the safe side.)
//   lookup_kernel: a workgroup stages all of W and walks all of it for its eight samples, with as many threads as it has
//   whatever K is, so its time goes with the rounds of workgroups (256 units, up to three on a unit as LDS allows) and jumps
//   at each.  Share of the general path's time (cached rows / others): D = 50, K = 64, three to a unit: 0.62 / 0.62 for the
//   6144 rows of one round, 0.75 to 0.9 / 0.99 in the second, 0.9 to 1.0 / 1.35 in the third; K = 512, one to a unit: 0.50 /
//   0.56 for 2048 rows, 0.88 / 0.95 in the second round, 1.2 / 1.2 and more in the third.  Wide rows whose W comes in several
//   pieces lose the second round (K = 2048, D = 50: 1.1 / 1.1); narrow ones (to 40 features: 0.95 to 1.05 / 1.0 at K =
//   1500, 0.8 / 0.75 at D = 16, K = 2048) win it, and where a round is shorter still beside the general path's launches the
//   third as well (D = 8, K = 4096: 0.82 / 0.72; the fourth 1.03 / 0.89).
//   small_kernel: the lanes per sample halve when the samples double (launch_small), so the time goes up in steps at powers
//   of two of the rows, and it works on whole groups of four features.  Rows and features rounded up so, times the nodes:
//   up to 5.5e8 it takes 0.7 to 0.99 of the general path's time on 256 to 4096 nodes, at 6.3e8 0.98 to 1.02, at 7.3e8 1.1 and
//   more (m K D alone put 5 features on 1024 nodes at 1.35).  Up to 128 nodes the general path's tiles are mostly
//   prologue and it stays behind on all of m K D <= kLWork (16 features: 0.81).
// (D < 4: the general path is the float32 search, slower than either up to m K D.)
static double look_up_rows(int K, int D)
{
    const double by_work = kLWork / ((double)K * D);
    if (D < 4) return by_work;
    if (lookup_in_lds(K, D)) return K <= 128 ? by_work : exp2(floor(log2(kLSteps / ((double)K * ((D + 3) / 4 * 4))))) - 1.0;
    const LookupLds l = lookup_lds(K, D);
    const int fit = (int)((size_t)160 * 1024 / (l.bytes + 1024)), pieces = (K + l.piece - 1) / l.piece;
    const int rounds = D <= 8 ? 3 : D <= 40 || pieces == 1 ? 2 : 1;
    const double by_rounds = 8.0 * 256 * rounds * (fit < 3 ? fit : 3);
    return by_work < by_rounds ? by_work : by_rounds;
}

// look-ups; qe (may be null) is overwritten.  Returns 1 when the call is not a small one.
int small_bmu_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, const float* W, int32_t K,
                  int32_t* bmu, float* d2, double* qe)
{
    if (ctx->search != SOM_SEARCH_AUTO || ctx->profiling || D > 64 || (double)m > look_up_rows(K, D)) return 1;
    SmallArgs a{};
    a.X = X;
    a.ldx = ldx;
    a.idx = idx;
    a.m = m;
    a.D = D;
    a.K = K;
    a.W = W;
    a.bmu = bmu;
    a.d2 = d2;
    a.qe_part = qe ? ctx->qe_part : nullptr;
    int rc;
    if (lookup_in_lds(K, D)) {
        rc = launch_small<false>(ctx, a, 2048);
    } else {
        const LookupLds l = lookup_lds(K, D);
        static bool attr_set_dev[kMaxDevices] = {};
        bool& attr_set = attr_set_dev[ctx->device];
        if (!attr_set) {
            for (const void* k : {reinterpret_cast<const void*>(lookup_kernel<4>), reinterpret_cast<const void*>(lookup_kernel<8>)})
                if (int e = check_hip(ctx, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSLds), "raising the dynamic LDS limit"))
                    return e;
            attr_set = true;
        }
        // (four samples a workgroup while that does not fill the chip: every workgroup reads all of W)
        if (m <= 4 * 256)
            hipLaunchKernelGGL(lookup_kernel<4>, dim3((unsigned)((m + 3) / 4)), dim3(kSThreads), l.bytes, ctx->stream, X, W, a, l.piece, l.stride);
        else
            hipLaunchKernelGGL(lookup_kernel<8>, dim3((unsigned)((m + 7) / 8)), dim3(kSThreads), l.bytes, ctx->stream, X, W, a, l.piece, l.stride);
        rc = check_hip(ctx, hipGetLastError(), "look-up kernel launch");
    }
    if (rc || !qe) return rc;
    hipLaunchKernelGGL(small_qe_kernel, dim3(1), dim3(kQeSlots), 0, ctx->stream, ctx->qe_part, qe);
    return check_hip(ctx, hipGetLastError(), "quantisation-error launch");
}

// a whole epoch without statistics.  Returns 1 when it is not a small one.
int small_epoch_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, float* W, int32_t K,
                    const float* G, double sigma, double eps_h)
{
    if (ctx->search != SOM_SEARCH_AUTO || ctx->profiling || ctx->reproducible || D > kSFeatures || K > kSNodes ||
        (double)m * K * D > kSWork || small_lds_bytes(K, D, true) > kSLds)
        return 1;
    // Two sets of sums take turns: this call's update clears the other one for the next call.  Under capture that would bake
    // one turn into the graph, and its replays would add to sums that nothing has cleared: a captured call clears the third
    // set with a launch of its own and leaves the turns alone.
    const size_t once = (size_t)K * (D + 1);
    const int copies = once * kSCopies <= kSCells ? kSCopies : 1;
    const size_t cells = once * copies;
    if (!ctx->small_sums) {
        if (hipMalloc((void**)&ctx->small_sums, 3 * kSCells * sizeof(double)) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the sums of a small map", 3 * kSCells * sizeof(double));
        }
        ctx->small_clean = 0;
    }
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (ctx->stream)                                            // (the null stream cannot be captured)
        if (int rc = check_hip(ctx, hipStreamIsCapturing(ctx->stream, &status), "capture status")) return rc;
    const bool captured = status != hipStreamCaptureStatusNone;
    const int turn = ctx->small_turn;
    double* const sums = ctx->small_sums + (captured ? 2 : turn) * kSCells;
    double* const next = captured ? nullptr : ctx->small_sums + (turn ^ 1) * kSCells;
    // (cells that are known to be zero in this call's set; a larger map than the last one clears its set first)
    if (captured || ctx->small_clean < cells)
        if (int rc = launch_fill_zero(ctx, sums, cells * sizeof(double))) return rc;
    SmallArgs a{};
    a.X = X;
    a.ldx = ldx;
    a.idx = idx;
    a.m = m;
    a.D = D;
    a.K = K;
    a.W = W;
    a.S = sums;
    a.copies = copies;
    if (!captured) ctx->small_clean = 0;                        // until this call's kernels are enqueued
    // (every workgroup adds its sums onto the map's: at most two per compute unit.  One each left a second pass to some of them:
    // 50,000 x 8 on 400 nodes 22.6 us instead of 18.8 to 20.5, 10^5 x 8 on 100 nodes 17.7 an epoch instead of 15.4)
    if (int rc = launch_small<true>(ctx, a, 512)) return rc;
    static bool attr_set_dev[kMaxDevices] = {};
    bool& attr_set = attr_set_dev[ctx->device];
    if (!attr_set) {
        if (int rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(small_update_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSLds),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    const double inv2s2 = 1.0 / (2.0 * sigma * sigma);
    const bool plain = ctx->eta == 1.0 && ctx->mu == 0.0;
    hipLaunchKernelGGL(small_update_kernel, dim3((unsigned)((K + kUNodes - 1) / kUNodes)), dim3(kUThreads), once * sizeof(double), ctx->stream,
                       G, sums, copies, K, D, inv2s2, ctx->safeguard == SOM_SAFEGUARD_SHIFT, eps_h, plain, ctx->eta, ctx->mu, ctx->velocity, W,
                       next);
    if (int rc = check_hip(ctx, hipGetLastError(), "small-map update launch")) return rc;
    if (!captured) {
        ctx->small_turn = turn ^ 1;
        ctx->small_clean = cells;
    }
    return SOM_OK;
}

} // namespace som
