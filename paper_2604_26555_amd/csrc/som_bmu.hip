// Best-matching-unit search for gfx950: fused score contraction + running arg-max, never storing N x K.
//
// For sample x and node k the kernel maximises  score(x, k) = x . w_k - |w_k|^2 / 2, which orders the nodes
// exactly as the squared distance |x - w_k|^2 = |x|^2 - 2 score does (paper Section 3.3.1: b(x) is the
// best-matching unit under the current weights).  The contraction runs as float32 MFMA
// (v_mfma_f32_32x32x2_f32): one instruction multiplies a 32-node x 2-feature slab of W by a 2-feature x 32-sample
// slab of X into a 32 x 32 block of scores, its accumulator pre-loaded with -|w_k|^2 / 2.
//
// Work split.  A wavefront owns MS blocks of 32 samples and keeps their features in registers for the whole
// kernel (lane l holds sample l % 32, features 2 s + l / 32).  The K nodes stream through LDS in stages of 128
// (double-buffered copies of padded weight rows), shared by the four wavefronts of a workgroup.  After each
// 32 x 32 block every lane folds its 16 scores into a running (best, runner-up, position) triple, so one lane
// only ever tracks the nodes of its own half of the rows; the two halves meet once at the end.  On this chip
// float32 MFMA and ordinary vector instructions occupy the same lanes (they do not overlap, not even across
// wavefronts), so the fold is held to four vector instructions per score.
//
// Exactness.  Scores are formed on centred values x - c, w - c (c = column means of W: distances are unchanged,
// magnitudes shrink to the spread of the map).  float32 accumulation leaves an error of at most
// (roundings) * 2^-24 * (|x - c| max|w - c| + max|w - c|^2 / 2) in a score, so a sample whose best two scores are
// closer than that worst-case bound is put on a list and re-decided by direct differences sum_d (x_d - w_kd)^2 on
// the values as given (lowest index wins ties): over every node (bmu_exact_kernel), or, for long lists, over the
// few nodes whose score lies inside the bound, which a second pass of the search collects (bmu_cand_kernel +
// bmu_cand_exact_kernel; the bf16 search for D <= 64 takes the differences at the end of its candidate tile, and knows the
// candidates of most of its near ties without that pass: pair_list).
// Where the caller asks for distances, the squared distance to the winner is formed by direct differences as well (in a
// stream over the rows of its own behind the bf16 searches), so the reported distances never carry the cancellation error of
// the score form.
//
// The default search (bmu_split_kernel further down for D <= 64, som_bmu_wide.hip above) is the same scheme with the
// contraction on the bf16 matrix pipe, samples and weights cut into two bf16 parts each.
#include "som_bmu_wide.hpp"

#include <math.h>

#include <type_traits>

namespace som {

constexpr int kWavesPerGroup = 4;
// Form of the split search's rows (D <= 64): whole 16-feature blocks of two bf16 parts; the packed block of four features alone;
// half-precision and fp6 parts of up to 32 features, and of up to 64.  kFormFew: rows as kFormWhole, four blocks of a map of up to
// kFewNodes nodes (scores are folded two at a time: bmu_split_tile).
enum SplitForm { kFormFew = -1, kFormWhole, kFormTail, kFormHalf1, kFormHalf2 };
constexpr int kFewNodes = 3 * kNodesPerStage;
constexpr int form_units(int form) { return form < kFormHalf1 ? 0 : form - kFormHalf1 + 1; }
// Scales of the half-precision parts: a sample's largest element comes to lie in [2^9, 2^10) (but the scale is at most twice the weights'), that
// of the nodes that the weights' scale is taken from in [2^2, 2^3), which leaves room for nodes 5800 times as far out.
constexpr int kHalfBit = 9, kHalfBitWeights = 2;
constexpr int kHalfRange = 28;         // most that the scales of samples lie below the weights'
constexpr int kHalfNorm = 14;          // the norms lie 2^14 below them,
constexpr float kHalfMost = 65504.0f;  // and fit half precision;
constexpr int kHalfThird = 10;         // the last of their three parts 2^10 less far
constexpr float kHalfNearest = 0.0625f;        // at the weights' scale: added to a node's norm where errors are charged for each unit of it
constexpr int half_norm_group(int D) { return (D + 3) / 4; }       // their place in the row, in fours: behind the features
__device__ __forceinline__ int half_scale(float most, int bit)
{
    const int e = bit + 127 - (int)(__float_as_uint(most) >> 23 & 255u);
    return e < -90 ? -90 : e > 90 ? 90 : e;
}
// the exponent of the fp6 scale that takes `most` into [3.75, 7.5]
__device__ __forceinline__ int fp6_scale(float most)
{
    const unsigned b = __float_as_uint(most);
    const int e = (int)(b >> 23 & 255u) - 129 + ((b & 0x7fffffu) > 0x700000u ? 1 : 0);
    return e < -40 ? -40 : e > 40 ? 40 : e;
}
constexpr int kThreads = kWavesPerGroup * 64;

constexpr uint32_t kCandMin = 4096;             // shortest list the candidate pass serves: its tiles take 15 to 30 us however few they are, the all-nodes
                                                // pass about 3.5 ns a sample (at K D = 51200); 6,000 entries on 400 nodes x 64: 18 + 13 us with it,
                                                // 5 + 55 without
constexpr uint32_t kCandMinFloat = 8192;        // the same of the float32 searches, whose tiles take about 40 us
constexpr uint32_t kCandHalfTiles = 65536;      // up to this length its tiles are halved (one per compute unit and more)
constexpr size_t kCandCapMax = (size_t)1 << 24; // longest one (bounds the candidate buffer at 512 MB + 64 MB)
constexpr int kCandGrid = 2048;
// Maps of fewer nodes send samples of more than four candidates to the candidate pass, whose time goes with the nodes; others keep up to eight.
// Candidate pass and pair list, 10^6 x 50 on 64 x 64 nodes close together: 197 + 56 us with four kept, 106 + 78 with eight; search on 1024 nodes 334 us
// and 326, 100,000 x 30 on 4096 141 and 134; but on 400 nodes (500,000 x 64) 23 + 18 and 23 + 20.
constexpr int kPairMany = 1024;
constexpr int kPairNodes = 65535;               // largest map whose node ids fit the pair list's 16-bit places (0xffff: none)

// floats of one 128-node stage (padded rows + half squared norms), rounded up to one float4 per thread
constexpr int stage_floats_for(int stride)
{
    return ((kNodesPerStage * (stride + 1) + 4 * kThreads - 1) / (4 * kThreads)) * (4 * kThreads);
}

// ---------------------------------------------------------------------------------------------------------
// Weight preparation: padded rows + half squared norms per (128-node stage, feature chunk), transposed copy,
// largest squared norm (scal[0], cleared beforehand), and the zeroing of the result words the later kernels count
// into.  A chunk holds stride - 1 features and one zero column (odd row stride); maps with D <= 64 have a single
// chunk.  One thread per element of the padded matrix (coalesced reads of W); the first kpad / 4 wavefronts also
// compute four nodes' norms each, in float64.
// ---------------------------------------------------------------------------------------------------------
// centre[f] = mean over nodes of W[k][f], f < D; zero up to the next multiple of 64.  Any vector would do (distances do not change when the same vector is
// taken off samples and weights); the mean keeps |w_k - centre| as small as the spread of the map.
__global__ void __launch_bounds__(1024) bmu_centre_kernel(const float* __restrict__ W, int K, int D, float* __restrict__ centre,
                                                          unsigned int* __restrict__ scal, float* __restrict__ spread, int32_t* __restrict__ small)
{
    stamp(small, kStampStart);
    __shared__ double part[16][64];
    __shared__ float ends[16][64][2];
    const int fl = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int f = blockIdx.x * 64 + fl;
    // this kernel runs first in every preparation: it also clears the result words (maximum norm, list lengths)
    if (blockIdx.x == 0 && threadIdx.x < 16) scal[threadIdx.x] = 0u;
    double s = 0.0;
    float low = INFINITY, high = -INFINITY;
    if (f < D) {
        // sixteen loads in flight per thread: the kernel is a chain of memory round trips otherwise
        int k = grp;
        for (; k + 15 * 16 < K; k += 16 * 16) {
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) v[u] = W[(size_t)(k + 16 * u) * D + f];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                s += (double)v[u];
                low = fminf(low, v[u]);
                high = fmaxf(high, v[u]);
            }
        }
        for (; k < K; k += 16) {
            const float v = W[(size_t)k * D + f];
            s += (double)v;
            low = fminf(low, v);
            high = fmaxf(high, v);
        }
    }
    part[grp][fl] = s;
    ends[grp][fl][0] = low;
    ends[grp][fl][1] = high;
    __syncthreads();
    if (grp == 0) {                       // the padding up to the next multiple of 64 entries is zeroed
        double t = 0.0;
        for (int q = 0; q < 16; ++q) t += part[q][fl];
        const float c = (f < D) ? (float)(t / K) : 0.0f;
        centre[f] = c;
        if (spread && blockIdx.x * 64 < (unsigned)D) {        // largest |w - centre| of these features
            for (int q = 0; q < 16; ++q) {
                low = fminf(low, ends[q][fl][0]);
                high = fmaxf(high, ends[q][fl][1]);
            }
            float most = f < D ? fmaxf(high - c, c - low) : 0.0f;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) most = fmaxf(most, __shfl_xor(most, o));
            if (fl == 0) spread[blockIdx.x] = most;
        }
    }
}

// The float32 search's stages (and any search's transposed copy, norms and maximum where the bf16 search does not apply).
__global__ void __launch_bounds__(256) bmu_prep_kernel(const float* __restrict__ W, int K, int D, int kpad, int stride,
                                                       int nch, int stage_floats, const float* __restrict__ centre,
                                                       float* __restrict__ stage, float* __restrict__ wt,
                                                       unsigned int* __restrict__ scal, double* __restrict__ qe,
                                                       int32_t* __restrict__ small)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    const int cols = nch * stride;
    if (e < 2 && qe) qe[e] = 0.0;
    if (e < 4 && small) small[e] = 0;
    if (e < kpad * cols) {
        const int k = e / cols, c = e - k * cols;
        const int ch = c / stride, fl = c - ch * stride;
        // stage column fl = 2 s + g feeds MFMA step s, half-wavefront g.  One chunk (D <= 64): feature fl.  Several
        // chunks: the lane's STEPS features are contiguous in a sample row, own range [first, first + STEPS) with
        // first = CH ch + STEPS g.  Where that range would run past D the lane reads the window [D - STEPS, D)
        // instead (always whole, always inside the row) and the columns in front of its own range hold zero
        // weights, so no feature is counted twice.
        const int steps = (stride - 1) / 2;
        const int first = ch * (stride - 1) + (fl & 1) * steps;
        const int window = first < D - steps ? first : D - steps;
        const int f = (nch == 1) ? fl : window + (fl >> 1);
        const bool own = fl < stride - 1 && f < D && (nch == 1 || f >= first);
        const bool real = k < K && own;
        const float v = real ? W[(size_t)k * D + f] : 0.0f;
        const int st = k / kNodesPerStage, r = k % kNodesPerStage;
        stage[((size_t)st * nch + ch) * stage_floats + (size_t)r * stride + fl] = real ? v - centre[f] : 0.0f;
    }
    // transposed copy, one thread per element with the node running fastest: coalesced writes (the reads, one row
    // apart, come from L2; written from the loop above the copy was 50,000 scattered 4-byte stores)
    if (e < D * kpad) {
        const int f = e / kpad, kk = e - f * kpad;
        wt[e] = (kk < K) ? W[(size_t)kk * D + f] : 0.0f;
    }
    // squared norm of the centred row exactly as the stage holds it (float32 differences), summed in float64: the
    // first kpad / 4 wavefronts of the grid take four nodes each (coalesced reads of their rows), and a workgroup
    // hands its largest norm to scal[0] with one atomic (one per node, all on the same word, took 10 us)
    __shared__ float wg_up[4];
    const int wv = e >> 6, lane = e & 63;
    float up_max = 0.0f;
    if (wv * 4 < kpad) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = wv * 4 + q;
            double nrm = 0.0;
            if (k < K)
                for (int f = lane; f < D; f += 64) {
                    const double v = (double)(W[(size_t)k * D + f] - centre[f]);
                    nrm += v * v;
                }
            nrm = wave_sum(nrm);
            if (lane == 0 && k < kpad) {
                const int st = k / kNodesPerStage, r = k % kNodesPerStage;
                const float nh = (k < K) ? (float)(-0.5 * nrm) : -INFINITY;
                for (int ch = 0; ch < nch; ++ch)
                    stage[((size_t)st * nch + ch) * stage_floats + (size_t)kNodesPerStage * stride + r] = nh;
                if (k < K) {
                    float up = (float)nrm;
                    if ((double)up < nrm) up = nextafterf(up, INFINITY);
                    up_max = fmaxf(up_max, up);
                }
            }
        }
    }
    if (lane == 0) wg_up[threadIdx.x >> 6] = up_max;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float m = fmaxf(fmaxf(wg_up[0], wg_up[1]), fmaxf(wg_up[2], wg_up[3]));
        if (m > 0.0f) atomicMax(&scal[0], __float_as_uint(m));
    }
}

// ---------------------------------------------------------------------------------------------------------
// Weight preparation of the bf16 search for D <= 64, one launch: a wavefront per node and lane per feature.
//   * Centre: the mean of up to kCentreNodes nodes, one from each stretch of K / kCentreNodes at a place that a hash of its number
//     picks, worked out by every workgroup for itself (any vector will do, the nearer to the middle of the weights the tighter
//     the bounds; a kernel of its own for the mean over all nodes cost 5 us and a launch).  Every (K / kCentreNodes)-th node
//     instead would be one or two columns of a lattice whose side divides that stride, off the middle: 10^6 x 50 on 64 x 64
//     nodes took 2.29 ms an epoch with those and takes 2.05 with these (shorter lists of near ties), on 32 x 32 0.452 and 0.448.
//   * Stage rows (layout at bmu_split_tile) are put together in LDS and leave it as whole lines, as do the sixteen nodes'
//     columns of the transposed copy; a plain copy of the rows in the stages' order serves the pair list.
//   * Packed tail (tail_r > 0): the last tail_r <= 4 features do not get a 16-feature block of their own (three MFMAs for a
//     block that is mostly padding) but one packed block whose sixteen slots hold the three products side by side,
//         weights  [ hi(r) | hi(r) | lo(r) | norm parts (3) | 0 ... ]   against samples  [ hi(r) | lo(r) | hi(r) | 1 1 1 | 0 ... ],
//     one MFMA.
//   * HALF: half-precision and fp6 parts instead (layout at bmu_split_tile; a wavefront's lanes trade them through its own part of LDS), the
//     norms' three parts in the places behind the features.  8.5 us at 1024 x 50, 6.2 with two bf16 parts.
//   * Norms: -|w|^2 / 2 + w . (w - hi - lo) behind the stage's rows (and as three bf16 parts in the packed block; the second term is what the
//     products of a sample that lies at the node drop), the largest norms of the nodes and of what the bf16 cut leaves over (w - hi,
//     w - hi - lo) in scal.
// Clears the result words that the later kernels of the call count into; the maxima it adds to (tops) were left zero by the
// re-decision of the call before.
// The sum over a wavefront, in every lane, by moves between lanes of the vector unit: four rotations within the rows of sixteen lanes, then the
// rows and the halves trade.  The preparation's four sums are a chain of steps that nothing runs beside; through LDS (__shfl_xor) a step waits for
// a round trip there: the kernel 6.9 us at 1024 x 50, 6.2 this way (437 x 37: 6.8 and 6.1).
template <int CTRL> __device__ __forceinline__ float rotated(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL> __device__ __forceinline__ double rotated(double x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)u, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
template <bool HALVES> __device__ __forceinline__ auto traded(unsigned x)
{
    if constexpr (HALVES) return __builtin_amdgcn_permlane32_swap(x, x, false, false);
    else return __builtin_amdgcn_permlane16_swap(x, x, false, false);
}
template <bool HALVES> __device__ __forceinline__ float both(float x)
{
    const auto r = traded<HALVES>(__float_as_uint(x));
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <bool HALVES> __device__ __forceinline__ double both(double x)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
    const auto lo = traded<HALVES>((unsigned)u), hi = traded<HALVES>((unsigned)(u >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (unsigned long long)hi[1] << 32 | lo[1]);
}
template <typename T> __device__ __forceinline__ T lanes_sum(T x)
{
    x += rotated<0x128>(x);
    x += rotated<0x124>(x);
    x += rotated<0x122>(x);
    x += rotated<0x121>(x);
    return both<true>(both<false>(x));
}

template <bool HALVES> __device__ __forceinline__ float larger(float x)
{
    const auto r = traded<HALVES>(__float_as_uint(x));
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float lanes_max(float x)
{
    x = fmaxf(x, rotated<0x128>(x));
    x = fmaxf(x, rotated<0x124>(x));
    x = fmaxf(x, rotated<0x122>(x));
    x = fmaxf(x, rotated<0x121>(x));
    return larger<true>(larger<false>(x));
}

constexpr int kCentreNodes = 64;
constexpr int kPrepNodes = 16;           // nodes (wavefronts) of a workgroup: 64 bytes of a row of the transposed copy

// a wavefront's writes to LDS before, its reads behind
__device__ __forceinline__ void wave_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

struct SplitPrep {
    char* stage16;
    float* wrow;
    int kb_count, tail_r, units, row_bytes, stage16_bytes;
};
struct HalfPrep : SplitPrep {};          // (half-precision and fp6 parts)

// the t-th of `count` nodes whose mean is the centre (count = K: all of them)
__device__ __forceinline__ int centre_node(int t, int count, int K)
{
    if (count == K) return t;
    uint32_t h = (uint32_t)t * 0x9e3779b1u;
    h ^= h >> 15;
    h *= 0x85ebca77u;
    h ^= h >> 13;
    return (int)((int64_t)t * K / count) + (int)__umulhi(h, (uint32_t)(K / count));
}

template <bool HALF>
__device__ __forceinline__ void split_prep(const float* __restrict__ W, int K, int D, int kpad, float* __restrict__ centre, float* __restrict__ wt,
                                           unsigned int* __restrict__ scal, unsigned int* __restrict__ tops, double* __restrict__ qe,
                                           int32_t* __restrict__ small, const SplitPrep& sp)
{
    __shared__ float part[kPrepNodes][64];
    __shared__ float given[kPrepNodes][65];
    __shared__ uint4 rows16[kPrepNodes * 272 / 16];           // [node][row_bytes]
    __shared__ float most[kPrepNodes][kTops];
    __shared__ __align__(16) _Float16 parts[HALF ? kPrepNodes : 1][2][64];          // HALF: first and second parts, by the places of a row
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int k0 = blockIdx.x * kPrepNodes, k = k0 + wave;           // rows of the stages (and of the transposed copy)
    stamp(small, kStampStart);
    if (blockIdx.x == 0) {
        if (tid < 16) scal[tid] = 0u;
        if (tid < 2 && qe) qe[tid] = 0.0;
        if (tid < 4 && small) small[tid] = 0;
    }
    __shared__ float spread[kPrepNodes];
    const bool real = k < K && lane < D;
    const float w = real ? W[(size_t)node_of_row(k, K) * D + lane] : 0.0f;
    const int count = K < kCentreNodes ? K : kCentreNodes;
    float v4[kCentreNodes / kPrepNodes];
#pragma unroll
    for (int u = 0; u < kCentreNodes / kPrepNodes; ++u) {
        const int t = wave * (kCentreNodes / kPrepNodes) + u;
        v4[u] = (t < count && lane < D) ? W[(size_t)centre_node(t, count, K) * D + lane] : 0.0f;
    }
    float s = 0.0f;
#pragma unroll
    for (int u = 0; u < kCentreNodes / kPrepNodes; ++u) s += v4[u];
    part[wave][lane] = s;
    if constexpr (HALF) {
        // how far the nodes of the centre lie from the first of them: the centre's own distances to within a factor of two
        const float v0 = lane < D ? W[(size_t)centre_node(0, count, K) * D + lane] : 0.0f;
        float top = 0.0f;
#pragma unroll
        for (int u = 0; u < kCentreNodes / kPrepNodes; ++u)
            top = fmaxf(top, wave * (kCentreNodes / kPrepNodes) + u < count ? fabsf(v4[u] - v0) : 0.0f);
        top = lanes_max(top);
        if (lane == 0) spread[wave] = top;
        parts[wave][0][lane] = (_Float16)0.0f;
        parts[wave][1][lane] = (_Float16)0.0f;
    }
    given[wave][lane] = w;
    for (int e = tid; e < kPrepNodes * sp.row_bytes / 16; e += 64 * kPrepNodes) rows16[e] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    float c = 0.0f;
#pragma unroll
    for (int u = 0; u < kPrepNodes; ++u) c += part[u][lane];
    c /= (float)count;                                        // zero behind the row
    if (blockIdx.x == 0 && wave == 0) centre[lane] = c;
    const float v = real ? w - c : 0.0f;
    char* const row = reinterpret_cast<char*>(rows16) + wave * sp.row_bytes;
    if constexpr (HALF) {
        // the scale: from the nodes that the centre is the mean of
        float top = spread[lane & (kPrepNodes - 1)];
        top = fmaxf(top, rotated<0x128>(top));
        top = fmaxf(top, rotated<0x124>(top));
        top = fmaxf(top, rotated<0x122>(top));
        top = fmaxf(top, rotated<0x121>(top));
        static_assert(kPrepNodes == 16, "a row of lanes");
        const int sw = half_scale(top, kHalfBitWeights);
        const float up = power_of_two(sw), back = power_of_two(-sw);
        if (blockIdx.x == 0 && tid == kScalShift) scal[kScalShift] = (unsigned)sw;
        // A node too far out for this scale has a row below all others, and the samples that may be near it are decided by direct
        // differences over all nodes.  (A weight that is no number stays: its scores are none either.)
        const double nrm = lanes_sum((double)v * (double)v);
        const bool out = 0.5 * nrm * (double)up * (double)up >= (double)(0.99f * kHalfMost) * (1 << kHalfNorm);
        const float h = out ? 0.0f : v * up;
        const _Float16 hi = (_Float16)h;
        const float left = h - (float)hi;
        // place of this lane's feature: features in fours, the last ones' window shifted back into the row (own features only, zeros in front)
        const int q = lane >> 2, start = 4 * q < D - 4 ? 4 * q : D - 4, slot = 4 * q + lane - start;
        if (real) {
            parts[wave][0][slot] = hi;
            parts[wave][1][slot] = (_Float16)left;
            reinterpret_cast<_Float16*>(row)[slot] = hi;
        }
        const float lo2 = lanes_sum(left * left);
        wave_lds();
        if (lane < 2 * sp.units) {
            const int u = lane >> 1, g = lane & 1;               // the first lane half feeds first parts, the other one second parts
            // (the order in which the tile's lanes come by a unit's values: its eights 0, 2, 1 and 3)
            uint4* from = reinterpret_cast<uint4*>(&parts[wave][g][32 * u]);
            struct {
                uint4 e[4];
            } eights = {{from[0], from[2], from[1], from[3]}};
            const halfx32 x = __builtin_bit_cast(halfx32, eights);
            const uintx16 pairs = __builtin_bit_cast(uintx16, eights);
            halfx2 big[4] = {};
#pragma unroll
            for (int i = 0; i < 16; ++i) big[i & 3] = __builtin_elementwise_max(big[i & 3], __builtin_bit_cast(halfx2, (unsigned int)pairs[i] & 0x7fff7fffu));
            big[0] = __builtin_elementwise_max(__builtin_elementwise_max(big[0], big[1]), __builtin_elementwise_max(big[2], big[3]));
            const int e = fp6_scale(fmaxf((float)big[0][0], (float)big[0][1]));
            const uintx6 p = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(x, power_of_two(e));
            const halfx32 d = __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(p, power_of_two(e));
            eights = __builtin_bit_cast(decltype(eights), d);
            from[0] = eights.e[0];
            from[2] = eights.e[1];
            from[1] = eights.e[2];
            from[3] = eights.e[3];
            char* const to = row + 32 * sp.kb_count;
            *reinterpret_cast<uint4*>(to + u * 32 + g * 16) = make_uint4(p[0], p[1], p[2], p[3]);
            *reinterpret_cast<uint2*>(to + sp.units * 32 + u * 16 + g * 8) = make_uint2(p[4], p[5]);
            reinterpret_cast<uint8_t*>(sp.stage16 + (size_t)(k / kNodesPerStage) * sp.stage16_bytes + (size_t)kNodesPerStage * (sp.row_bytes + 4))
                [4 * (k % kNodesPerStage) + 2 * g + u] = (uint8_t)(127 + e);
        }
        wave_lds();
        const float off_hi = real ? (float)hi - (float)parts[wave][0][slot] : 0.0f, off_lo = real ? left - (float)parts[wave][1][slot] : 0.0f;
        const float off_hi2 = lanes_sum(off_hi * off_hi), off_lo2 = lanes_sum(off_lo * off_lo),
                    with_rest = lanes_sum(v * (off_lo * back));
        if (lane == 0) {
            const double full = -0.5 * nrm + (double)with_rest;
            const float nh = (float)full;
            reinterpret_cast<float*>(sp.stage16 + (size_t)(k / kNodesPerStage) * sp.stage16_bytes +
                                     (size_t)kNodesPerStage * sp.row_bytes)[k % kNodesPerStage] = (k < K && nh > kSplitPadNorm) ? nh : kSplitPadNorm;
            // three parts (11 bits each) of the norm at 2^-kHalfNorm of its scale, which meet that factor on the samples' side (the last
            // one, which may be as small as half precision goes, at 2^kHalfThird of theirs), and what keeps padding rows below all others
            const float at = (float)(full * (double)up * (double)up * (1.0 / (1 << kHalfNorm)));
            _Float16* cell = reinterpret_cast<_Float16*>(row) + 4 * half_norm_group(D);
            const _Float16 p0 = (_Float16)at, p1 = (_Float16)(at - (float)p0), p2 = (_Float16)(((at - (float)p0) - (float)p1) * (float)(1 << kHalfThird));
            const _Float16 least = (_Float16)-kHalfMost;
            const bool own = k < K && !out;
            cell[0] = own ? p0 : least;
            cell[1] = own ? p1 : least;
            cell[2] = own ? p2 : least;
            cell[3] = own ? (_Float16)0.0f : least;
            float most2 = (float)nrm;
            if ((double)most2 < nrm) most2 = nextafterf(most2, INFINITY);
            most[wave][0] = k < K ? most2 : 0.0f;
            // Norms of what the parts leave over, as they are and for each unit of the node's own (and kHalfNearest): a bound charges two nodes
            // theirs, not twice the farthest one's.
            const float norm = sqrtf(most2), per = own ? 1.0f / (norm + kHalfNearest * back) : 0.0f;
            const float over[3] = {sqrtf(lo2) * back, sqrtf(off_hi2) * back, sqrtf(off_lo2) * back};
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                most[wave][1 + t] = over[t] * per;
                most[wave][4 + t] = own ? over[t] : 0.0f;
            }
            // the nearest of the nodes that are too far out: how far its bits lie below those of infinity
            most[wave][7] = k < K && out ? __uint_as_float(0x7f800000u - __float_as_uint(norm * 0.999999f)) : 0.0f;
        }
    } else {
        const __bf16 hi = (__bf16)v;
        const float left = v - (float)hi;
        const __bf16 lo = (__bf16)left;
        const float rest = left - (float)lo;
        const double nrm = lanes_sum((double)v * (double)v);
        const float lo2 = lanes_sum(left * left), rest2 = lanes_sum(rest * rest), with_rest = lanes_sum(v * rest);
        if (real) {
            const int tail0 = D - sp.tail_r;
            if (lane < tail0) {
                // slot group q = four features, its window [min(4 q, D - 4), + 4): own elements only, zeros in front of them
                const int q = lane >> 2, start = 4 * q < D - 4 ? 4 * q : D - 4;
                const int kb = q >> 2, g = (q >> 1) & 1, t = (q & 1) * 4 + lane - start;
                __bf16* cell = reinterpret_cast<__bf16*>(row + kb * 64 + g * 32) + t;
                cell[0] = hi;
                cell[8] = lo;
            } else {
                __bf16* cell = reinterpret_cast<__bf16*>(row + sp.kb_count * 64) + (lane - tail0);
                cell[0] = hi;
                cell[sp.tail_r] = hi;
                cell[2 * sp.tail_r] = lo;
            }
        }
        if (lane == 0) {
            const float nh = (float)(-0.5 * nrm + (double)with_rest);
            const float nf = (k < K && nh > kSplitPadNorm) ? nh : kSplitPadNorm;
            reinterpret_cast<float*>(sp.stage16 + (size_t)(k / kNodesPerStage) * sp.stage16_bytes +
                                     (size_t)kNodesPerStage * sp.row_bytes)[k % kNodesPerStage] = nf;
            if (sp.tail_r) {
                // cut into three bf16 parts (exactly: 3 x 8 bits), which meet ones on the samples' side
                const __bf16 p0 = (__bf16)nf;
                const __bf16 p1 = (__bf16)(nf - (float)p0);
                const __bf16 p2 = (__bf16)((nf - (float)p0) - (float)p1);
                __bf16* cell = reinterpret_cast<__bf16*>(row + sp.kb_count * 64) + 3 * sp.tail_r;
                cell[0] = p0;
                cell[1] = p1;
                cell[2] = p2;
            }
            float up = (float)nrm;
            if ((double)up < nrm) up = nextafterf(up, INFINITY);
            most[wave][0] = k < K ? up : 0.0f;
            most[wave][1] = lo2;
            most[wave][2] = rest2;
        }
    }
    __syncthreads();
    // sixteen rows of a stage are contiguous (kNodesPerStage is a multiple of sixteen)
    uint4* to = reinterpret_cast<uint4*>(sp.stage16 + (size_t)(k0 / kNodesPerStage) * sp.stage16_bytes + (size_t)(k0 % kNodesPerStage) * sp.row_bytes);
    for (int e = tid; e < kPrepNodes * sp.row_bytes / 16; e += 64 * kPrepNodes) to[e] = rows16[e];
    const int f = tid >> 4, q = tid & 15;
    if (f < D) wt[(size_t)f * kpad + k0 + q] = given[q][f];
    if (real) sp.wrow[(size_t)k * D + lane] = w;
    if (tid < (HALF ? kTops : 3)) {
        float m = most[0][tid];
        for (int u = 1; u < kPrepNodes; ++u) m = fmaxf(m, most[u][tid]);
        if (m > 0.0f) atomicMax(&tops[tid], __float_as_uint(m));
    }
}

__global__ void __launch_bounds__(64 * kPrepNodes) bmu_split_prep_kernel(const float* __restrict__ W, int K, int D, int kpad,
                                                                         float* __restrict__ centre, float* __restrict__ wt,
                                                                         unsigned int* __restrict__ scal, unsigned int* __restrict__ tops,
                                                                         double* __restrict__ qe, int32_t* __restrict__ small, const SplitPrep sp)
{
    split_prep<false>(W, K, D, kpad, centre, wt, scal, tops, qe, small, sp);
}
__global__ void __launch_bounds__(64 * kPrepNodes) bmu_split_prep_kernel(const float* __restrict__ W, int K, int D, int kpad,
                                                                         float* __restrict__ centre, float* __restrict__ wt,
                                                                         unsigned int* __restrict__ scal, unsigned int* __restrict__ tops,
                                                                         double* __restrict__ qe, int32_t* __restrict__ small, const HalfPrep sp)
{
    split_prep<true>(W, K, D, kpad, centre, wt, scal, tops, qe, small, sp);
}

__global__ void fill_zero_kernel(uint32_t* p, size_t words)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < words; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// ---------------------------------------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------------------------------------

// The re-decision list of a pass.  The search kernels do not append to it themselves: one atomic per wavefront on the
// list's single length word serialises in the memory system (about 10 ns each; with a few per cent of the samples
// listed nearly every wavefront has one, and the 15,625 wavefronts of 10^6 samples then spent up to 0.1 ms of a
// 0.4 ms kernel queueing for it).  Each sample instead gets one word, its cut (best score minus the rounding bound)
// or kNotListed, and this kernel compacts the listed ones: a workgroup takes 4096 samples at a time, counts with a
// scan, and reserves its entries with one atomic.  The order of the list is immaterial (every entry is decided on its
// own).
constexpr int kListThreads = 1024, kListPerThread = 4;

__global__ void __launch_bounds__(kListThreads) bmu_list_kernel(const BmuArgs a)
{
    __shared__ unsigned int wave_base[2][kListThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int64_t per_block = (int64_t)kListThreads * kListPerThread;
    for (int64_t chunk = blockIdx.x; chunk * per_block < a.m; chunk += gridDim.x) {
        const int64_t i0 = chunk * per_block + (int64_t)tid * kListPerThread;
        float c[kListPerThread];
        if (i0 + kListPerThread <= a.m) {
            const float4 t = *reinterpret_cast<const float4*>(a.cut_all + i0);      // i0 is a multiple of four
            c[0] = t.x;
            c[1] = t.y;
            c[2] = t.z;
            c[3] = t.w;
        } else {
#pragma unroll
            for (int q = 0; q < kListPerThread; ++q) c[q] = (i0 + q < a.m) ? a.cut_all[i0 + q] : kNotListed;
        }
        static_assert(kListPerThread == 4, "a thread's cuts travel as one float4");
        unsigned int mine = 0u;                            // entries of the list below, entries of the pair list above bit 16
#pragma unroll
        for (int q = 0; q < kListPerThread; ++q) mine += (c[q] == kPairs) ? 0x10000u : (c[q] == c[q]) ? 1u : 0u;
        unsigned int incl = mine;                         // inclusive scan over the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int t = __shfl_up(incl, o);
            if (lane >= o) incl += t;
        }
        if (lane == 63) wave_base[0][wave] = incl;
        __syncthreads();
        if (wave == 0) {
            // exclusive scan of the wavefronts' totals; the last lane reserves the workgroup's entries
            const unsigned int w = lane < kListThreads / 64 ? wave_base[0][lane] : 0u;
            unsigned int wi = w;
#pragma unroll
            for (int o = 1; o < kListThreads / 64; o <<= 1) {
                const unsigned int t = __shfl_up(wi, o);
                if (lane >= o) wi += t;
            }
            const unsigned int total = __shfl(wi, kListThreads / 64 - 1);
            // both lists' lengths are neighbours: one atomic reserves the entries of both
            unsigned long long base = 0ull;
            if (lane == 0 && total)
                base = atomicAdd(reinterpret_cast<unsigned long long*>(&a.scal[a.slot]),
                                 (unsigned long long)(total & 0xffffu) | ((unsigned long long)(total >> 16) << 32));
            const unsigned int base0 = __shfl((unsigned int)base, 0), base1 = __shfl((unsigned int)(base >> 32), 0);
            if (lane < kListThreads / 64) {
                wave_base[0][lane] = base0 + ((wi - w) & 0xffffu);
                wave_base[1][lane] = base1 + ((wi - w) >> 16);
            }
        }
        __syncthreads();
        const unsigned int before = incl - mine;
        unsigned int pos = wave_base[0][wave] + (before & 0xffffu), pos1 = wave_base[1][wave] + (before >> 16);
#pragma unroll
        for (int q = 0; q < kListPerThread; ++q) {
            if (c[q] == kPairs) {
                a.recheck_end[-1 - (int64_t)pos1] = (uint32_t)(i0 + q);
                ++pos1;
            } else if (c[q] == c[q]) {
                a.recheck[pos] = (uint32_t)(i0 + q);
                a.cutv[pos] = c[q];
                ++pos;
            }
        }
        __syncthreads();                                 // wave_base is rewritten by the next chunk
    }
}

// Up to seven 16-bit node ids and their count in 128 bits of registers.  A hit shifts the ids up by one place (the
// oldest drops out at the top, the count keeps counting, so an overflow shows): no memory traffic while the scores
// are being formed, one 16-byte store per lane at the end.
struct CandSet {
    unsigned long long lo = 0ull, hi = 0ull;
    int n = 0;
    // id = base + off
    __device__ __forceinline__ void note(int base, int off)
    {
        // (The empty statement keeps the branch that skips these instructions when no lane of the wavefront has a
        // hit, which is four times out of five: without it the compiler runs them under an empty mask, and every
        // vector instruction here is paid for in matrix time.  Passing the base through it keeps the addition
        // inside the skipped region as well.)
        asm volatile("" : "+v"(base));
        const int id = base + off;
        hi = (hi << 16) | (lo >> 48);
        lo = (lo << 16) | (unsigned long long)(unsigned int)id;
        ++n;
    }
    __device__ __forceinline__ ulonglong2 packed() const
    {
        const unsigned long long c = (unsigned long long)(n < 0xffff ? n : 0xffff);
        return make_ulonglong2(lo, (hi & 0xffffffffffffull) | (c << 48));
    }
};
__device__ __forceinline__ int cand_count(const ulonglong2& v) { return (int)(v.y >> 48); }
__device__ __forceinline__ int cand_id(const ulonglong2& v, int t)
{
    return (int)(((t < 4) ? (v.x >> (16 * t)) : (v.y >> (16 * (t - 4)))) & 0xffffull);
}

// ---------------------------------------------------------------------------------------------------------
// main kernel
// ---------------------------------------------------------------------------------------------------------
// One tile = the kWavesPerGroup * MS * 32 samples of a workgroup against all nodes.
// CAND = false: the search proper (samples wave0 ..., running best / runner-up, results and list at the end).
// CAND = true: the candidate pass over the first `count` entries of the re-decision list: the same scores are
// formed again, and instead of the fold every score that reaches the entry's cut is noted (node id into the
// lane's own slots: lane (j, g) sees the nodes of half g only, so no two lanes share a slot and no atomics are
// needed).  One compare per score instead of four fold instructions.
// PAD = true: the last stage ends in whole blocks of padding nodes (K is at least 32 short of a multiple of 128),
// which are skipped; a variant of its own so that the stage body of the other maps stays one basic block.
template <int STEPS, int MS, bool CAND, bool PAD = false>
__device__ __forceinline__ void bmu_tile(const BmuArgs& a, int64_t first, int64_t tile_index, unsigned int count,
                                         float4* lds4)
{
    constexpr int STRIDE = 2 * STEPS + 1;
    constexpr int STAGE_FLOATS = stage_floats_for(STRIDE);   // whole float4s per thread: no tail handling
    constexpr int STAGE_F4 = STAGE_FLOATS / 4;
    constexpr int PRE = STAGE_F4 / kThreads;
    float* lds = reinterpret_cast<float*>(lds4);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int j = lane & 31;
    const int g = lane >> 5;
    const int64_t wave0 = first + (tile_index * kWavesPerGroup + wave) * (MS * 32);   // first = position of tile 0

    // centre[2 s + g]: both candidates are read through wave-uniform addresses (scalar loads), the lane picks one
    // (the array is zero-padded to a multiple of 64 entries, so no index needs a bound)
    auto centre_of = [&](int s) {
        const float c0 = a.centre[2 * s], c1 = a.centre[2 * s + 1];
        return g ? c1 : c0;
    };

    // ---- this wavefront's samples, kept in registers
    float x[MS][STEPS];
    bool valid[MS];
    float cut[MS];          // CAND
    CandSet noted[MS];      // CAND
    // (Staging the workgroup's rows through LDS with coalesced 16-byte loads was measured against this direct
    // gather and lost by 3 to 10 %: the gather is served by the vector L1, the staging adds two barriers.)
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
        int64_t i = wave0 + mb * 32 + j;
        const int64_t total = CAND ? (int64_t)count : a.m;
        valid[mb] = i < total;
        int64_t ii = valid[mb] ? i : total - 1;
        if constexpr (CAND) {
            cut[mb] = valid[mb] ? a.cutv[ii] : NAN;     // no score compares >= NaN
            ii = (int64_t)a.recheck[ii];
        }
        const int64_t row = a.idx ? (int64_t)a.idx[ii] : ii;
        const float* xr = a.X + row * a.ldx;
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            const int f = 2 * s + g;
            // Unconditional load through a clamped index.  Beyond D the value is a copy of the last feature; it
            // meets zero weights in the stage rows, and the epilogue masks it out of the norms.
            x[mb][s] = xr[f < a.D ? f : a.D - 1];
        }
    }

    // running best / runner-up scores of this lane's half of the rows, and where the best one sits
    float best[MS], second[MS];
    int rsel[MS], tsel[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
        best[mb] = -INFINITY;
        second[mb] = -INFINITY;
        rsel[mb] = 0;
        tsel[mb] = 0;
    }

    // ---- stream the nodes through LDS
    const int nstages = a.kpad / kNodesPerStage;
    const float4* src4 = reinterpret_cast<const float4*>(a.stage);
    {
        float4 first[PRE];
#pragma unroll
        for (int p = 0; p < PRE; ++p) first[p] = src4[tid + p * kThreads];
        // the samples are centred only now, with the first stage's loads already on their way
#pragma unroll
        for (int mb = 0; mb < MS; ++mb)
#pragma unroll
            for (int s = 0; s < STEPS; ++s) x[mb][s] -= centre_of(s);
#pragma unroll
        for (int p = 0; p < PRE; ++p) lds4[tid + p * kThreads] = first[p];
    }
    __syncthreads();

    for (int st = 0; st < nstages; ++st) {
        const int buf = st & 1;
        // the next stage travels global -> registers now and registers -> LDS after this stage's arithmetic
        // (the last iteration reloads its own stage into the idle buffer, which keeps the loop branch-free).
        // Named scalars rather than an array, and a scheduling fence behind the loads: otherwise the compiler
        // sinks every load to its use after the MFMAs and the copy is no longer hidden.
        float4 pre0, pre1, pre2, pre3, pre4, pre5, pre6, pre7, pre8;
        static_assert(PRE <= 9, "stage copy holds at most nine float4 per thread");
        {
            const int nxt = (st + 1 < nstages) ? st + 1 : st;
            const float4* s4 = src4 + (size_t)nxt * STAGE_F4 + tid;
#define SOM_PRE_LOAD(i) if constexpr (PRE > i) pre##i = s4[i * kThreads];
            SOM_PRE_LOAD(0) SOM_PRE_LOAD(1) SOM_PRE_LOAD(2) SOM_PRE_LOAD(3) SOM_PRE_LOAD(4)
            SOM_PRE_LOAD(5) SOM_PRE_LOAD(6) SOM_PRE_LOAD(7) SOM_PRE_LOAD(8)
#undef SOM_PRE_LOAD
        }
        __builtin_amdgcn_sched_barrier(0);
        const float* wbuf = lds + buf * STAGE_FLOATS;
        const float* nbuf = wbuf + kNodesPerStage * STRIDE;

        // Fully unrolled: with the stage body in one basic block the prefetch loads above stay ahead of the MFMAs.
        // The LDS reads of node block nb + 1 (weights and -|w|^2/2) are written into the MFMA sequence of block nb,
        // one read per pair of MFMAs, and pinned there: left alone the scheduler sometimes gathers all reads of a
        // block in front of its first MFMA, and the matrix pipe then idles for an LDS round trip per block.
        float wa[STEPS];
        floatx16 c;
        {
            const float* wrow = wbuf + j * STRIDE + g;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) wa[s] = wrow[2 * s];
            const float4* nh = reinterpret_cast<const float4*>(nbuf + 4 * g);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 t = nh[2 * q];
                c[4 * q + 0] = t.x;
                c[4 * q + 1] = t.y;
                c[4 * q + 2] = t.z;
                c[4 * q + 3] = t.w;
            }
        }
#pragma unroll
        for (int nb = 0; nb < kNodesPerStage / 32; ++nb) {
            constexpr int NB = kNodesPerStage / 32;
            if constexpr (PAD) {
                if (st * kNodesPerStage + nb * 32 >= a.K) break;           // padding from here to the end of the stage
            }
            const int nx = (nb + 1 < NB) ? nb + 1 : nb;                    // the last block re-reads itself (unused)
            const float* wnext = wbuf + (nx * 32 + j) * STRIDE + g;
            const float4* nhnext = reinterpret_cast<const float4*>(nbuf + nx * 32 + 4 * g);
            float wn[STEPS];
            floatx16 cn;
            floatx16 acc[MS];
#pragma unroll
            for (int mb = 0; mb < MS; ++mb) acc[mb] = c;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
#pragma unroll
                for (int mb = 0; mb < MS; ++mb)
                    acc[mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(wa[s], x[mb][s], acc[mb], 0, 0, 0);
                if (nb + 1 < NB) {
                    wn[s] = wnext[2 * s];
                    if (s < 4) {
                        const float4 t = nhnext[2 * s];
                        cn[4 * s + 0] = t.x;
                        cn[4 * s + 1] = t.y;
                        cn[4 * s + 2] = t.z;
                        cn[4 * s + 3] = t.w;
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, MS, 0);    // MS MFMAs
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // one LDS read
                }
            }
            const int tile = st * (kNodesPerStage / 32) + nb;
            if constexpr (CAND) {
#pragma unroll
                for (int mb = 0; mb < MS; ++mb) {
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (acc[mb][r] >= cut[mb]) noted[mb].note(tile * 32 + 4 * g, 8 * (r >> 2) + (r & 3));
                }
            }
            // fold the 16 scores of each block into the running triple: four VALU instructions per score
#pragma unroll
            for (int mb = 0; mb < (CAND ? 0 : MS); ++mb) {
                const float before = best[mb];
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float v = acc[mb][r];
                    rsel[mb] = (v > best[mb]) ? r : rsel[mb];
                    second[mb] = __builtin_amdgcn_fmed3f(best[mb], second[mb], v);
                    best[mb] = vmax(best[mb], v);
                }
                tsel[mb] = (best[mb] > before) ? tile : tsel[mb];
            }
            if (nb + 1 < NB) {
#pragma unroll
                for (int s = 0; s < STEPS; ++s) wa[s] = wn[s];
                c = cn;
            }
        }

        {
            float4* d4 = lds4 + (buf ^ 1) * STAGE_F4 + tid;
#define SOM_PRE_STORE(i) if constexpr (PRE > i) d4[i * kThreads] = pre##i;
            SOM_PRE_STORE(0) SOM_PRE_STORE(1) SOM_PRE_STORE(2) SOM_PRE_STORE(3) SOM_PRE_STORE(4)
            SOM_PRE_STORE(5) SOM_PRE_STORE(6) SOM_PRE_STORE(7) SOM_PRE_STORE(8)
#undef SOM_PRE_STORE
        }
        __syncthreads();
    }

    if constexpr (CAND) {
#pragma unroll
        for (int mb = 0; mb < MS; ++mb)
            if (valid[mb])
                a.cand[(size_t)(wave0 + mb * 32 + j) * 2 + g] = noted[mb].packed();
        return;
    }
    // ---- join the two half-wavefronts, then lane (j, g) finishes block mp + g
    const float wmax2 = __uint_as_float(a.scal[0]);
    const float wmax = sqrtf(wmax2) * 1.000001f;
    // two scores, each with two roundings per MFMA step (k = 2) and one in -|w|^2/2; the roundings of x - centre
    // and w - centre move a score difference by at most 2 and 4 more units: (4 STEPS + 8) * 2^-24, plus slack
    const float rel = (float)(4 * STEPS + 12) * 5.9604645e-08f;
    double qs = 0.0, qs2 = 0.0;
#pragma unroll
    for (int mp = 0; mp < MS; mp += 2) {
        float r_best = 0.f, r_second = 0.f, r_xn = 0.f, r_part = 0.f;
        int r_node = 0;
        bool r_valid = false;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int mb = mp + q;
            if (mb >= MS) break;
            int node = tsel[mb] * 32 + 8 * (rsel[mb] >> 2) + 4 * g + (rsel[mb] & 3);
            const float ob = __shfl_xor(best[mb], 32);
            const float os = __shfl_xor(second[mb], 32);
            const int on = __shfl_xor(node, 32);
            const float sec = fmaxf(fmaxf(second[mb], os), fminf(best[mb], ob));
            const bool other = (ob > best[mb]) || (ob == best[mb] && on < node);
            const float bst = other ? ob : best[mb];
            node = other ? on : node;
            node = node < a.K ? node : a.K - 1;
            // squared norm of the centred sample and squared distance to the winner (both centred the same way),
            // half the features per lane
            // (the winner's centred weights come from its stage row, which holds them in this lane's order with
            // zeros beyond D: no centring and no bounds here)
            float xn = 0.f, part = 0.f;
            const float* wr = a.stage + (size_t)(node / kNodesPerStage) * STAGE_FLOATS +
                              (size_t)(node % kNodesPerStage) * STRIDE + g;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                const float xm = (2 * s + g < a.D) ? x[mb][s] : 0.0f;
                const float df = xm - wr[2 * s];
                xn = fmaf(xm, xm, xn);
                part = fmaf(df, df, part);
            }
            xn += __shfl_xor(xn, 32);
            part += __shfl_xor(part, 32);
            if (q == g) {
                r_best = bst;
                r_second = sec;
                r_node = node;
                r_xn = xn;
                r_part = part;
                r_valid = valid[mb];
            }
        }
        const int64_t i = wave0 + (mp + g) * 32 + j;
        // magnitude bound of every partial sum of the score: |w|^2/2 + |sum x_d w_d| <= |w|^2/2 + |x| |w|
        const float xl = sqrtf(r_xn);
        const float bound = (xl * wmax + 0.5f * wmax2) * rel;
        // the two centring roundings leave an error of 2^-23 d (|x| + |w|) in d^2: hand the few samples that
        // sit within 2^-9 (|x| + |w|) of their node to the exact pass, which works on the values as given
        const float tiny = (xl + wmax) * (xl + wmax) * 3.8146973e-06f;
        const bool close = r_valid && a.K > 1 && (!((r_best - r_second) > bound) || r_part < tiny);
        if (r_valid) {
            a.bmu[i] = r_node;
            if (a.d2) a.d2[i] = r_part;
            if (!close) {
                qs += sqrt((double)r_part);
                qs2 += (double)r_part;
            }
        }
        if (r_valid) a.cut_all[i] = close ? list_cut(r_best - bound) : kNotListed;
    }
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

// two workgroups per compute unit (LDS-bound), i.e. two wavefronts per SIMD: the register budget is 256 VGPRs
template <int STEPS, int MS, bool PAD>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    // The first full_tiles workgroups take MS blocks per wavefront; the rest of the grid, the last partial round
    // of the launch, takes tiles of half that size, which spread more evenly over the compute units.
    if ((int64_t)blockIdx.x < a.full_tiles) {
        bmu_tile<STEPS, MS, false, PAD>(a, 0, blockIdx.x, 0u, lds4);
    } else if constexpr (MS > 1) {
        constexpr int64_t per_full = (int64_t)kWavesPerGroup * MS * 32;
        bmu_tile<STEPS, MS / 2, false, PAD>(a, a.full_tiles * per_full, (int64_t)blockIdx.x - a.full_tiles, 0u, lds4);
    }
}

// true when this call's list is long enough for the candidate pass to pay and fits its buffers (device-side: the
// host does not know the list length)
__device__ __forceinline__ bool cand_pass_serves(const BmuArgs& a, unsigned int count)
{
    return count > a.cand_min && count <= a.cand_cap;
}

// candidate pass: a fixed grid walks the tiles of the list
template <int STEPS, int MS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_cand_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    const unsigned int count = a.scal[a.slot];
    if (!cand_pass_serves(a, count)) return;
    constexpr int64_t per_tile = (int64_t)kWavesPerGroup * MS * 32;
    if constexpr (MS > 1) {
        // a list that leaves compute units idle goes through in tiles of half the size: twice as many workgroups,
        // each done in half the time
        if (count <= kCandHalfTiles) {
            for (int64_t t = blockIdx.x; t * (per_tile / 2) < (int64_t)count; t += gridDim.x)
                bmu_tile<STEPS, MS / 2, true>(a, 0, t, count, lds4);
            return;
        }
    }
    for (int64_t t = blockIdx.x; t * per_tile < (int64_t)count; t += gridDim.x) bmu_tile<STEPS, MS, true>(a, 0, t, count, lds4);
}

// ---------------------------------------------------------------------------------------------------------
// The same search with the contraction on the bf16 matrix pipe (this kernel: 4 <= D <= 64, som_bmu_wide.hip: D > 64; the default for every map of more than one node).
//
// A float32 value v is cut into two bf16 parts, hi = bf16(v) and lo = bf16(v - hi) (both rounded to nearest, the
// difference is exact in float32), so that |v - lo - hi| <= 2^-16 |v| (2^-8 from each part's eight significant bits).  A score then
// takes three bf16 MFMAs per 16 features (v_mfma_f32_32x32x16_bf16, products exact, float32 accumulation):
//     x . w  ~  xh . wh + xl . wh + xh . wl,
// the dropped parts together below 3 * 2^-16 |x| |w|.  The bf16 pipe runs these three in 96 cycles where the
// float32 MFMAs of the same 16 features take 512, and unlike those it leaves three quarters of the vector issue
// slots to the fold, which runs beside it.  Nothing else changes: the error bound is wider (the split, and the pipe's
// accumulation error per MFMA, charged as any-order float32 summation), samples inside it go on the same list and are decided by the same direct
// differences, so the results are those of the float32 search.
//
// Layout.  Lane (j, g) of a wavefront holds, for k-block kb, the eight features of slot groups q = 4 kb + 2 g and
// q + 1, group q being the window [min(4 q, D - 4), + 4) of the row: always whole and inside the row, so a group is
// one 16-byte load; where the window is shifted back the stage rows hold zero weights in front of the group's own
// features, and no feature is counted twice.  A stage row is [kb][g][hi x 8 | lo x 8] bf16 plus 16 bytes of padding
// (row stride 64 * blocks + 16 bytes: the 16-byte reads of sixteen consecutive rows fall into distinct banks), followed
// by the stage's 128 half squared norms in float32.
// Half-precision and fp6 parts (HALF; large calls of 21 to 64 features: half_parts_pay).  A value is cut into its half-precision part and what
// that leaves over; a score takes the product of the first parts on v_mfma_f32_32x32x16_f16 and both cross products from fp6 copies of the parts
// in one v_mfma_scale_f32_32x32x64_f8f6f4 for 32 features ([second | first] against [first | second], as in som_bmu_held.hip): 4 + 2
// MFMAs a block at 50 features where two bf16 parts take 10.  The norms travel as three half-precision parts in the four places behind the
// features, against a factor on the samples' side; the fourth keeps padding rows below all others.  A sample is scaled by the power of
// two of its largest element, the weights by one that 64 of them give, and each node's 32 features have
// an fp6 scale of their own in LDS behind the norms.  Nodes up to some 5800 times as far out as those 64 fit (kHalfBitWeights); of one farther
// still no score is formed, and only samples at least half as far out are decided over all nodes.  10^6 x 50 on 1024 nodes, one of them 100, 1000
// or 10,000 times as far out: search 240 us, as without it (two bf16 parts 309, 344 and 966).  Errors are charged by the norms of the nodes
// that come into question: with the largest over all nodes such a node would widen every sample's bound.  The bound is about 2.2 times that of two bf16 parts (fp6 has four significant bits:
// |first - fp6| |second| and its mirror image for each of the two scores compared), so about twice as many samples are listed.
// 10^6 x 50: search on 1024 nodes 292 -> 242 us, on 4096 1070 -> 814; with the longer lists the epochs took 414 -> 372 and 1340 -> 1211 us.
// What bounds it: the port that issues vector instructions and MFMAs (41 and 6 a block of 32 x 32, the matrix pipe busy 0.45 to 0.55 of the
// time at 1.8 to 2.0 GHz).  Third and fourth fp6 products (what fp6 leaves of the first parts) would bring the bound back to that of bf16 for 7 or
// 8 MFMAs a block: an estimated 7 % of the search for what the lists would give back; not built.
// The fold takes a class's scores four at a time: two medians meet the runner-up in one v_max3 (10 vector instructions for four scores
// until then, 9 now; 838 -> 814 us of search on 4096 nodes).
// The fold keeps the position inside a block in the low four bits of the score (one and-or instead of a compare
// and a select; 16 units of the last place are part of the bound), so padding nodes carry a large finite negative
// norm here instead of -inf.
// ---------------------------------------------------------------------------------------------------------
// bytes of a stage row.  bf16 parts: kb whole 16-feature blocks of 64 bytes, 32 bytes for a packed tail block, 16 bytes of padding.
// Half-precision and fp6 parts: 32 bytes a 16-feature block, 48 bytes 32 features, an odd number of sixteens.
constexpr int split_row_bytes(int kb, int form)
{
    return form_units(form) ? (kb * 32 + form_units(form) * 48) / 16 * 16 + ((kb * 2 + form_units(form) * 3) % 2 ? 0 : 16)
                            : kb * 64 + (form == kFormTail ? 32 : 0) + 16;
}
// (behind the rows 128 norms, and with fp6 parts their scales: a byte for each half and unit)
constexpr int split_stage_f4(int kb, int form)
{
    return ((kNodesPerStage * split_row_bytes(kb, form) + kNodesPerStage * (form_units(form) ? 8 : 4)) / 16 + kThreads - 1) / kThreads * kThreads;
}
// Stages go from memory to LDS directly (DIRECT: no registers, no vector instructions for it) where two of them lie below 64 KB, in whole
// kilobytes; others by way of registers: four whole blocks of two bf16 parts (53 to 64 features) and half-precision parts of 61 to 64.
// Search of 10^6 x 50 on 4096 nodes 814 us by registers and 754, on 1024 242 and 225; of 10^7 x 50 on 1024 2212 and 2123.  The first stage is
// asked for before the samples are: behind their cutting it was waited for in full, which on small maps is much of a tile (10^6 rows on 100
// nodes, 50 features 71.6 us by registers, 72.9 with the first stage asked for late, 64.6 early; 20 features 45.2, 44.6, 43.7; 900,000 x 25 on 400
// nodes 84.5, 80.7, 80.5; 1024 and 4096 nodes the same).
constexpr int split_pitch_direct(int kb, int form)
{
    return (kNodesPerStage * split_row_bytes(kb, form) + kNodesPerStage * (form_units(form) ? 8 : 4) + 1023) / 1024 * 1024;
}
constexpr bool split_direct(int kb, int form) { return 2 * split_pitch_direct(kb, form) <= 64512; }        // (a kilobyte for what lies in front)
// bytes from one stage to the next in LDS
constexpr int split_pitch(int kb, int form) { return split_direct(kb, form) ? split_pitch_direct(kb, form) : split_stage_f4(kb, form) * 16; }
constexpr int kSplitMinNodes = 1;              // SOM_SEARCH_AUTO: every map of more than this many nodes (measured faster than the
                                               // float32 search from 2 x 2 nodes and from D = 4 on)
constexpr int kSplitMS = 2;

// The candidate pass: what a wavefront keeps in LDS behind the stages.  A lane whose scores of a block reach its sample's cut adds one
// entry (which of its sixteen rows, the sample, the block) to the wavefront's queue; the direct differences are taken from the queue,
// a lane an entry, so that lanes share the work whosever samples' it is, and the nearest candidate of each sample is kept as the
// least (distance, node) in one 64-bit word.  (With up to seven ids in each lane's registers, every lane walked the longest
// set of its wavefront, and samples with more went to the all-nodes pass.)  10^6 x 50 on
// 64 x 64 nodes, 254,000 entries: pass and all-nodes pass 430 + 284 us then, 352 + 23 with the queue.
struct CandQueue {
    static constexpr size_t kFixed = 64 * (sizeof(unsigned long long) + sizeof(uint32_t));
    unsigned long long* nearest;     // [64] per sample of the tile
    uint32_t* row;                   // [64] its row of X
    uint2* entry;                    // [kQueue]
};
constexpr int cand_queue(int kb, int form)            // entries; two workgroups fit a compute unit
{
    const size_t left = (80 * 1024 - 2 * (size_t)split_pitch(kb, form)) / kWavesPerGroup - CandQueue::kFixed;
    return left / sizeof(uint2) < 512 ? (int)(left / sizeof(uint2)) / 16 * 16 : 512;
}
constexpr size_t cand_lds(int kb, int form)
{
    return 2 * (size_t)split_pitch(kb, form) + kWavesPerGroup * (CandQueue::kFixed + (size_t)cand_queue(kb, form) * sizeof(uint2));
}

// first feature of slot group q (four consecutive features)
__device__ __forceinline__ int split_window(int q, int D) { return 4 * q < D - 4 ? 4 * q : D - 4; }

// CAND = true: the candidate pass over the first `count` entries of the re-decision list (as in bmu_tile): the same
// scores are formed again, bit for bit, and every node whose score reaches the entry's cut is noted.
// KB whole 16-feature blocks (three MFMAs each) and, with TAIL, one packed block for the last a.tail_r <= 4 features
// (one MFMA; layout at bmu_split_prep_kernel).
// first feature of lane half g's h-th window of k-block kb: only the last block of a row without a packed tail can be shifted
template <int KB, int FORM>
__device__ __forceinline__ int split_start(int kb, int g, int h, int D)
{
    return kb < KB - (form_units(FORM) ? 2 : 1) ? 16 * kb + 8 * g + 4 * h : split_window(4 * kb + 2 * g + h, D);
}

// A lane's part of the rows of MS sample blocks, as given.
template <int KB, int FORM, int MS, bool CAND>
struct SplitRows {
    static constexpr bool TAIL = FORM == kFormTail;
    static constexpr int LOADED = form_units(FORM) && KB > 2 * form_units(FORM) ? KB - 1 : KB;      // (a last block that holds the norms only)
    float4 x[MS][KB > 0 ? KB : 1][2], t[MS];

    __device__ __forceinline__ void load(const BmuArgs& a, int64_t wave0, int64_t total, int j, int g)
    {
#pragma unroll
        for (int mb = 0; mb < MS; ++mb) {
            int64_t ii = wave0 + mb * 32 + j;
            ii = ii < total ? ii : total - 1;
            if constexpr (CAND) ii = (int64_t)a.recheck[ii];
            const float* xr = a.X + (a.idx ? (int64_t)a.idx[ii] : ii) * a.ldx;
#pragma unroll
            for (int kb = 0; kb < LOADED; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) x[mb][kb][h] = load4(xr + split_start<KB, FORM>(kb, g, h, a.D));
            if constexpr (TAIL) t[mb] = load4(xr + a.D - 4);         // (inside the row: D >= 4)
        }
    }
};

// A lane's operands of a node block: whole blocks' first and second bf16 parts, the packed block and the norms; or half-precision parts, fp6 parts and
// the scales of those.
template <int KB, int FORM>
struct SplitFragments {
    static constexpr bool TAIL = FORM == kFormTail;
    static constexpr int H = form_units(FORM), KBA = KB > 0 ? KB : 1;
    bf16x8 wh[KBA], wl[KBA], wtl;
    floatx16 c;
    halfx8 half[KBA];
    uintx6 q[H > 0 ? H : 1];
    int scales;

    __device__ __forceinline__ void read_half(int kb, const char* row) { half[kb] = *reinterpret_cast<const halfx8*>(row + 32 * kb); }
    __device__ __forceinline__ void read_fp6(int u, const char* row, int g)
    {
        const uint4 t = *reinterpret_cast<const uint4*>(row + 32 * KB + 32 * u);
        const uint2 r = *reinterpret_cast<const uint2*>(row + 32 * KB + 32 * H + 16 * u - 8 * g);         // (row carries g * 16)
        q[u][0] = t.x;
        q[u][1] = t.y;
        q[u][2] = t.z;
        q[u][3] = t.w;
        q[u][4] = r.x;
        q[u][5] = r.y;
    }
    __device__ __forceinline__ void first(const char* row, const char* tail, int g)
    {
        if constexpr (H > 0) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) read_half(kb, row);
#pragma unroll
            for (int u = 0; u < H; ++u) read_fp6(u, row, g);
            scales = *reinterpret_cast<const uint16_t*>(tail);
        } else {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                wh[kb] = *reinterpret_cast<const bf16x8*>(row + kb * 64);
                wl[kb] = *reinterpret_cast<const bf16x8*>(row + kb * 64 + 16);
            }
            if constexpr (TAIL) wtl = *reinterpret_cast<const bf16x8*>(row + KB * 64 - g * 16);
            const float4* nh = reinterpret_cast<const float4*>(tail);
#pragma unroll
            for (int n = 0; n < 4; ++n) {
                const float4 t = TAIL ? float4{0.f, 0.f, 0.f, 0.f} : nh[2 * n];
                c[4 * n + 0] = t.x;
                c[4 * n + 1] = t.y;
                c[4 * n + 2] = t.z;
                c[4 * n + 3] = t.w;
            }
        }
    }
};

// the two halves of a wavefront trade: a keeps its lower half's values and takes b's in its upper half, b the others
__device__ __forceinline__ void swap_halves(float& a, float& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(int& a, int& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    a = (int)r[0];
    b = (int)r[1];
}

template <int KB, int FORM, int MS, bool CAND>
__device__ __forceinline__ void bmu_split_tile(const BmuArgs& a, int64_t first, int64_t tile_index, unsigned int count,
                                               float4* lds4)
{
    constexpr bool TAIL = FORM == kFormTail;
    constexpr int H = form_units(FORM), HA = H > 0 ? H : 1;
    constexpr bool HALF = H > 0;
    constexpr bool FOUR = FORM != kFormFew;            // scores are folded four at a time, otherwise two (below)
    constexpr int RS = split_row_bytes(KB, FORM);
    constexpr int STAGE_F4 = split_stage_f4(KB, FORM);
    constexpr int KBA = KB > 0 ? KB : 1;               // array lengths (no zero-length arrays when D <= 4)
    constexpr int PRE = STAGE_F4 / kThreads;
    constexpr bool DIRECT = split_direct(KB, FORM);
    constexpr int PITCH = split_pitch(KB, FORM);
    const char* ldsb = reinterpret_cast<const char*>(lds4);

    const int tid = threadIdx.x;
    int lane = tid & 63;
    if constexpr (CAND) asm volatile("" : "+v"(lane));
    const int wave = tid >> 6;
    const int j = lane & 31;
    const int g = lane >> 5;
    const int64_t wave0 = first + (tile_index * kWavesPerGroup + wave) * (MS * 32);

    // ---- this wavefront's samples: centred, cut into bf16 parts, kept in registers
    bf16x8 xh[MS][KBA], xl[MS][KBA], xt[MS];
    // search: norm of the centred sample (both lane halves hold the whole row's), what a score errs by for each unit of |w| and besides
    // (err_w, err_0), and the norm of what the cut leaves over (see below); HALF: err_w, the norms of that, of the second part and of what
    // fp6 leaves of the first, and the scale of the scores.  They wait in LDS, behind the stages, for the end of the
    // tile: the stage loop has no registers to spare for them.
    float* const stash = reinterpret_cast<float*>(lds4 + 2 * PITCH / 16) + threadIdx.x;
    float cut[MS];          // CAND
    unsigned int found[MS]; // CAND: hits of the block in hand
    const int64_t total = CAND ? (int64_t)count : a.m;
    // DIRECT: a stage's kilobytes from memory to LDS, a stretch of them for each wavefront
    const float4* src4 = reinterpret_cast<const float4*>(a.stage16);
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char*)lds4);
    const int wave_s = __builtin_amdgcn_readfirstlane(wave);
    auto load_stage = [&](int st, int buf) {
        constexpr int KBYTES = PITCH / 1024, PER = (KBYTES + kWavesPerGroup - 1) / kWavesPerGroup;
        const char* from = reinterpret_cast<const char*>(src4) + (size_t)st * STAGE_F4 * 16 + wave_s * (PER * 1024);
        const unsigned to = lds0 + (unsigned)(buf * PITCH + wave_s * (PER * 1024));
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (wave_s * PER + q < KBYTES) lds_load16(from + q * 1024, (unsigned)lane * 16u, to + q * 1024);
    };
    // (the first stage is on its way while the samples come in and are cut: nobody has read or written this buffer yet, or not since the
    // barrier between two tiles; by registers too: 10^6 x 64 on 100 nodes 89 us behind the cut and 85)
    if constexpr (DIRECT) {
        load_stage(0, 0);
    } else {
#pragma unroll
        for (int p = 0; p < PRE; ++p) lds4[tid + p * kThreads] = src4[tid + p * kThreads];
    }
    SplitRows<KB, FORM, MS, CAND> raw;
    raw.load(a, wave0, total, j, g);
    // CAND: the wavefront's queue, its length (which may pass the end: those entries are lost, and lost remembers whose), and each
    // sample's row
    constexpr int QUEUE = cand_queue(KB, FORM);
    CandQueue cq{};
    unsigned int queued = 0u, lost = 0u;
    if constexpr (CAND) {
        char* at = reinterpret_cast<char*>(lds4 + 2 * PITCH / 16) + wave * (CandQueue::kFixed + QUEUE * sizeof(uint2));
        cq.nearest = reinterpret_cast<unsigned long long*>(at);
        cq.entry = reinterpret_cast<uint2*>(at + 64 * sizeof(unsigned long long));
        cq.row = reinterpret_cast<uint32_t*>(at + 64 * sizeof(unsigned long long) + QUEUE * sizeof(uint2));
#pragma unroll
        for (int mb = 0; mb < MS; ++mb) {
            const int64_t i = wave0 + mb * 32 + j;
            cut[mb] = i < total ? a.cutv[i] : NAN;       // no score compares >= NaN
            cut[mb] = cut[mb] > -INFINITY ? cut[mb] : NAN;      // (a row without a cut: to the all-nodes pass)
            found[mb] = 0u;
            const uint32_t is = a.recheck[i < total ? i : total - 1];
            if (g == 0) {
                cq.row[mb * 32 + j] = a.idx ? a.idx[is] : is;
                cq.nearest[mb * 32 + j] = ~0ull;
            }
        }
    }
    // HALF: the half-precision parts' fragments, the fp6 parts', and their scales (a byte for each unit)
    halfx8 xf[MS][KBA];
    uintx6 xq[MS][HA];
    int xs[MS];
    const int sw = HALF ? (int)a.scal[kScalShift] : 0;
    if constexpr (HALF) {
#pragma unroll
        for (int mb = 0; mb < MS; ++mb) {
            constexpr int LOADED = SplitRows<KB, FORM, MS, CAND>::LOADED;
            float v[LOADED][8], most = 0.0f;
#pragma unroll
            for (int kb = 0; kb < LOADED; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int at = 16 * kb + 8 * g + 4 * h, start = split_start<KB, FORM>(kb, g, h, a.D);
                    const float4 cen = load4(a.centre + start), x4 = raw.x[mb][kb][h];
                    float* to = &v[kb][4 * h];
                    to[0] = x4.x - cen.x;
                    to[1] = x4.y - cen.y;
                    to[2] = x4.z - cen.z;
                    to[3] = x4.w - cen.w;
                    if (kb >= KB - 2) {            // (windows shifted back: own elements only)
                        const int shift = at - start;
#pragma unroll
                        for (int t = 0; t < 4; ++t) to[t] = shift <= t ? to[t] : 0.0f;
                    }
                    most = fmaxf(most, fmaxf(fmaxf(fabsf(to[0]), fabsf(to[1])), fmaxf(fabsf(to[2]), fabsf(to[3]))));
                }
            float other = most;
            swap_halves(most, other);
            most = fmaxf(most, other);
            // The sample's scale: its largest element into [2^9, 2^10), unless that leaves what the norms' factor can hold (elements past what half
            // precision holds make the bound infinite: such a sample goes to the all-nodes pass).
            int sx = half_scale(most, kHalfBit);
            sx = sx < sw - kHalfRange ? sw - kHalfRange : sx > sw + 1 ? sw + 1 : sx;
            const float s = power_of_two(sx), back = power_of_two(-sx);
            // scales of the fp6 parts: second parts are at most a half unit of the largest element's first part (lanes 0 to 31 pack them)
            const int eh = (int)(__float_as_uint(most * s) >> 23) - 129, eq = g == 0 ? eh - 12 : eh;
            const int e = eq < -40 ? -40 : eq > 40 ? 40 : eq;
            const float q_scale = power_of_two(e);
            xs[mb] = (127 + e) * 0x101;
            float v2 = 0.0f, e2 = 0.0f, after2 = 0.0f;
#pragma unroll
            for (int u = 0; u < H; ++u) {
                unsigned int hi[8], lo[8];
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int kb = 2 * u + (t >> 2);
                    hi[t] = lo[t] = 0u;
                    if (kb < LOADED) {
                        const HalfPair h(v[kb < LOADED ? kb : 0][2 * (t & 3)] * s, v[kb < LOADED ? kb : 0][2 * (t & 3) + 1] * s);
                        hi[t] = h.hi;
                        lo[t] = h.lo;
                    }
                }
                xf[mb][2 * u] = __builtin_bit_cast(halfx8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
                if (2 * u + 1 < KB) xf[mb][2 * u + 1 < KB ? 2 * u + 1 : 0] = __builtin_bit_cast(halfx8, make_uint4(hi[4], hi[5], hi[6], hi[7]));
                // the first lane half packs the second parts of all thirty-two features, the other half the first parts
                uintx16 w;
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    unsigned int m = lo[t], n = hi[t];
                    swap_words(m, n);
                    w[t] = m;
                    w[8 + t] = n;
                }
                const uintx6 q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(__builtin_bit_cast(halfx32, w), q_scale);
                xq[mb][u] = q;
                if constexpr (!CAND) {
                    const uintx16 d = __builtin_bit_cast(uintx16, __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(q, q_scale));
                    float s2[2] = {0.0f, 0.0f};
#pragma unroll
                    for (int t = 0; t < 16; ++t) {
                        const halfx2 o = __builtin_bit_cast(halfx2, (unsigned int)w[t]);
                        const halfx2 r = o - __builtin_bit_cast(halfx2, (unsigned int)d[t]);
                        s2[(t >> 2) & 1] = __builtin_amdgcn_fdot2(o, o, s2[(t >> 2) & 1], false);
                        e2 = __builtin_amdgcn_fdot2(r, r, e2, false);
                    }
                    v2 += s2[0] + s2[1];
                    const float after = (float)(KB - 2 * u);          // MFMAs of first parts from its own on
                    after2 = fmaf(after * after, s2[0], fmaf((after - 1.0f) * (after - 1.0f), s2[1], after2));
                }
            }
            if constexpr (KB > 2 * H) xf[mb][KB - 1] = __builtin_bit_cast(halfx8, make_uint4(0u, 0u, 0u, 0u));
            {
                // the norms' factor, 2^(kHalfNorm + sx - sw), twice, 2^-kHalfThird of it (which may be subnormal), and 2^15 (padding rows)
                const unsigned int f = (unsigned)(15 + kHalfNorm + sx - sw) << 10;
                const int third = 15 + kHalfNorm - kHalfThird + sx - sw;
                static_assert(15 + kHalfNorm - kHalfThird - kHalfRange >= -9, "2^-24 at least");
                const unsigned int f2 = third >= 1 ? (unsigned)third << 10 : 1u << (9 + third);
                const int group = half_norm_group(a.D);
                const uint4 w = __builtin_bit_cast(uint4, xf[mb][KB - 1]);
                const bool here = ((group >> 1) & 1) == g, second = (group & 1) != 0;
                const unsigned int f0 = here ? f | f << 16 : 0u, f1 = here ? f2 | 0x7800u << 16 : 0u;
                xf[mb][KB - 1] = __builtin_bit_cast(halfx8, make_uint4(w.x | (second ? 0u : f0), w.y | (second ? 0u : f1), w.z | (second ? f0 : 0u),
                                                                       w.w | (second ? f1 : 0u)));
            }
            if constexpr (!CAND) {
                // The error of a score.  (1) What the cuts drop: with x = xh + xl, ql and qh the fp6 copies of the parts, and w likewise, a score misses
                // (xl - ql) . wh + ql . (wh - qh_w) + xh . (wl - ql_w) + (xh - qh) . ql_w + xl . wl.  Two scores are compared, so the first
                // counts by wh_a - wh_b; of the third the preparation gives w . (wl - ql_w) back, which leaves (x - w) . (wl - ql_w) and
                // xl . (wl - ql_w).  All norms are formed; the weights' are the largest over the nodes for each unit of |w| (and
                // kHalfNearest).  (A second part is rounded to half precision before it goes to fp6, and a subnormal part costs what 2^-14
                // would: 2^-25 at the sample's scale, a feature.)
                // (2) The pipe's accumulation: an MFMA of first parts is charged sixteen units of its accumulator and products
                // (any order of its additions), those of fp6 products sixty-four terms each; they go first and hold small numbers
                // only.  Block kb of the first parts is in the accumulator of KB - kb MFMAs, the norm in that of the last.
                // (3) Six units for the roundings of the two centrings and of -|w|^2 / 2, and what its third part can lose: 2^-25 of the
                // weights' scale, 2^(kHalfNorm - kHalfThird) times.
                float h2 = v2, eh2 = e2, ha2 = after2;               // lower lanes: second parts; upper lanes: first parts
                swap_halves(v2, h2);
                swap_halves(e2, eh2);
                swap_halves(after2, ha2);
                auto root = [&](float x) { return __builtin_amdgcn_sqrtf(x + kSquaresFloor) * (1.001f * back); };
                constexpr float unit = 5.9604645e-08f, small = 80.0f * (H + 2) * unit;
                const float nh = root(h2), least = 2.5e-7f * back;            // 2^-25 in each of 64 features
                const float nl = root(v2) * 1.001f + least, nx = nh + nl;
                const float nr = root(e2) + nl * 4.9e-4f + least, qh = root(eh2);
                const float err_w = root(ha2) * (16.3f * unit) + nl * small + nx * (6.0f * unit);
                if (MS == 1 || mb == g) {
                    stash[0] = nx;
                    stash[kThreads] = err_w;
                    stash[2 * kThreads] = nr * 1.001f;
                    stash[3 * kThreads] = nl * 1.001f;
                    stash[4 * kThreads] = qh * 1.001f;
                    stash[5 * kThreads] = __int_as_float(sx + sw);
                }
            }
        }
    }
    const int tail_r = TAIL ? a.tail_r : 0;
    // The packed block (layout at bmu_split_prep_kernel): slot s of the sixteen holds copy s / tail_r of tail feature s % tail_r,
    // the samples' copies being hi, lo, hi (against the weights' hi, hi, lo), then three ones.  A lane's four words (slots 8 g to
    // 8 g + 7) are put together from the window [D - 4, D) by byte permutations: which bytes of the four hi and of the four
    // lo parts, and the ones.
    unsigned int tail_sel[4][3];
    if constexpr (TAIL) {
        auto choose = [&](auto r_) {
            constexpr int r = decltype(r_)::value;
#pragma unroll
            for (int w = 0; w < 4; ++w)
#pragma unroll
                for (int part = 0; part < 3; ++part) {
                    constexpr auto sel = [](int gg, int w_, int part_) {
                        unsigned int out = 0u;
                        for (int h = 0; h < 2; ++h) {
                            const int slot = 8 * gg + 2 * w_ + h, copy = slot / r;
                            const unsigned at = 2u * (unsigned)(4 - r + slot % r);
                            const bool hit = part_ == 2 ? (slot >= 3 * r && slot < 3 * r + 3) : (copy < 3 && (copy == 1) == (part_ == 1));
                            const unsigned v = part_ == 2 ? (hit ? 0x3f80u : 0u) : hit ? (at | ((at + 1u) << 8)) : 0x0c0cu;
                            out |= v << (16 * h);
                        }
                        return out;
                    };
                    tail_sel[w][part] = g == 0 ? sel(0, w, part) : sel(1, w, part);
                }
        };
        if (tail_r == 1) choose(std::integral_constant<int, 1>{});
        else if (tail_r == 2) choose(std::integral_constant<int, 2>{});
        else if (tail_r == 3) choose(std::integral_constant<int, 3>{});
        else choose(std::integral_constant<int, 4>{});
    }
#pragma unroll
    for (int mb = 0; mb < (HALF ? 0 : MS); ++mb) {
        // squares: of the first parts, the same weighted by how many of the large MFMAs follow (xa), of the second parts (lo2) and
        // of what both leave over (rest2)
        float hi2 = 0.0f, xa = 0.0f, lo2 = 0.0f, rest2 = 0.0f;
        if constexpr (TAIL) {
            const float4 cen = load4(a.centre + a.D - 4);
            const float4 v4 = raw.t[mb];
            // (elements in front of the tail belong to the whole blocks)
            const float v[4] = {tail_r > 3 ? v4.x - cen.x : 0.0f, tail_r > 2 ? v4.y - cen.y : 0.0f, tail_r > 1 ? v4.z - cen.z : 0.0f, v4.w - cen.w};
            unsigned int h[2], l[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const SplitPair p(v[2 * q], v[2 * q + 1]);
                if constexpr (!CAND) {
                    hi2 = square2(p.hi, hi2);
                    lo2 = square2(p.lo, lo2);
                    rest2 = p.rest2(rest2);
                }
                h[q] = p.hi;
                l[q] = p.lo;
            }
            // (both lane halves hold the tail's features: they count once)
            hi2 = g == 0 ? hi2 : 0.0f;
            lo2 = g == 0 ? lo2 : 0.0f;
            rest2 = g == 0 ? rest2 : 0.0f;
            xa = hi2;
            uint4 out;
            out.x = __builtin_amdgcn_perm(h[1], h[0], tail_sel[0][0]) | __builtin_amdgcn_perm(l[1], l[0], tail_sel[0][1]) | tail_sel[0][2];
            out.y = __builtin_amdgcn_perm(h[1], h[0], tail_sel[1][0]) | __builtin_amdgcn_perm(l[1], l[0], tail_sel[1][1]) | tail_sel[1][2];
            out.z = __builtin_amdgcn_perm(h[1], h[0], tail_sel[2][0]) | __builtin_amdgcn_perm(l[1], l[0], tail_sel[2][1]) | tail_sel[2][2];
            out.w = __builtin_amdgcn_perm(h[1], h[0], tail_sel[3][0]) | __builtin_amdgcn_perm(l[1], l[0], tail_sel[3][1]) | tail_sel[3][2];
            xt[mb] = __builtin_bit_cast(bf16x8, out);
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            float v[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int q = 4 * kb + 2 * g + h, start = split_start<KB, FORM>(kb, g, h, a.D);
                const float4 cen = load4(a.centre + start), x4 = raw.x[mb][kb][h];
                v[4 * h + 0] = x4.x - cen.x;
                v[4 * h + 1] = x4.y - cen.y;
                v[4 * h + 2] = x4.z - cen.z;
                v[4 * h + 3] = x4.w - cen.w;
                if (!TAIL && kb == KB - 1) {
                    // (slots in front of a shifted window's own features read zero: they meet zero weights in the stage rows, and
                    // stay out of the norms)
                    const int shift = 4 * q - start;
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[4 * h + t] = shift <= t ? v[4 * h + t] : 0.0f;
                }
            }
            if constexpr (CAND) {
                split8(v, xh[mb][kb], xl[mb][kb]);
            } else {
                float s8 = 0.0f;
                split8(v, xh[mb][kb], xl[mb][kb], s8, lo2, rest2);
                constexpr float after = (float)(KB + (TAIL ? 1 : 0));
                hi2 += s8;
                xa = fmaf((after - (float)kb) * (after - (float)kb), s8, xa);
            }
        }
        if constexpr (!CAND) {
            // The error of a score, in three parts.  (1) What the bf16 cut drops: with x = xh + xl + xr and w likewise,
            // xl . wl + xr . w + (x - xr) . wr, of which the preparation gives w . wr back.  Two scores are compared, so what counts is by how
            // much their errors differ: |xl| |wl| each, |xr| |w_a - w_b|, and |x - w| |wr| and |xr| |wr| each, where neither of the two
            // nodes is farther from the sample than the winner is, nor from each other than twice that (nor than both norms).  The largest
            // |w - wh| and |wr| over the nodes come from the weight preparation: norms that were formed (a part has eight significant
            // bits, so the worst case is 3 * 2^-16 |x| |w|, several times more).  With |w_a| + |w_b| and |x| in the places of the
            // distances, as before, a map of 1024 nodes along a chain had 38 % of 10^7 x 50 rows listed and has 28 %, one of 64 x 64 48 % of
            // 10^6 and 40 %.
            // (2) The pipe's accumulation.  How an MFMA orders and rounds the additions of its sixteen exact products to its
            // accumulator C is not documented, so each MFMA is charged what seventeen float32 terms can lose when added in
            // ANY order with one rounding to nearest per addition: 16 * 2^-24 (|C| + sum |products|).  (The largest error seen on
            // operands built against aligning, truncating and sequential adders stays well inside 16 units:
            // tests/test_gpu_matrix_pipe.py fails on the first result outside them.)  The small products (lo hi, hi lo) go first,
            // into accumulators that hold nothing else, so they are charged for their own size; the large ones (hi hi) of block kb
            // are in the accumulator of the KB - kb (+ 1 with a tail) MFMAs from their own on, which the weighted norm xa adds up.
            // Half squared norms: in the accumulator of all 3 KB MFMAs, or of the packed block's only.
            // (3) Six units for the roundings of the two centrings and of -|w|^2 / 2.
            hi2 += __shfl_xor(hi2, 32);
            xa += __shfl_xor(xa, 32);
            lo2 += __shfl_xor(lo2, 32);
            rest2 += __shfl_xor(rest2, 32);
            const float lo_w = __builtin_amdgcn_sqrtf(__uint_as_float(a.norms[1]) + kSquaresFloor) * 1.001f;
            const float rest_w = __builtin_amdgcn_sqrtf(__uint_as_float(a.norms[2]) + kSquaresFloor) * 1.001f;
            // |xl| (before its own cut) and |x| are at most what their parts add up to
            const float nr = __builtin_amdgcn_sqrtf(rest2 + kSquaresFloor) * 1.0001f;
            const float nl = __builtin_amdgcn_sqrtf(lo2 + kSquaresFloor) * 1.0001f + nr, nh = __builtin_amdgcn_sqrtf(hi2 + kSquaresFloor) * 1.0001f;
            const float nx = nh + nl;
            constexpr float unit = 5.9604645e-08f;
            const float err_w = nl * (32.64f * KB * unit) + __builtin_amdgcn_sqrtf(xa + kSquaresFloor) * (1.0001f * 16.256f * unit) + nx * (6.0f * unit);
            // (lane (j, g) finishes sample j of block g)
            if (MS == 1 || mb == g) {
                stash[0] = nx;
                stash[kThreads] = nl * lo_w * 1.0078125f + nr * rest_w * 1.0078125f + nx * lo_w * (32.64f * KB * unit);
                // (two figures of sixteen bits, rounded up: LDS is full)
                stash[2 * kThreads] =
                    __uint_as_float(((__float_as_uint(err_w) + 0xffffu) & 0xffff0000u) | ((__float_as_uint(nr * 1.0078125f) + 0xffffu) >> 16));
            }
        }
    }

    // Running best / runner-up scores (position in the block in the low bits of the score) and the block the best one came
    // from, for each of four classes of nodes: even and odd rows of the block, even and odd blocks.  Nodes that lie next to
    // each other on the map, whose scores are the ones that come close, mostly fall into different classes (with the two lane
    // halves: eight), so that a near tie is mostly one between class winners, whose ids are known at the end of the tile.
    // Four sets instead of one cost registers, but no more fold instructions than the block numbers' updates.
    constexpr int CLS = CAND ? 1 : 4;
    float best[MS][CLS], second[MS][CLS], before[MS][CLS];
    int tsel[MS][CLS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
#pragma unroll
        for (int c = 0; c < CLS; ++c) {
            best[mb][c] = -INFINITY;
            second[mb][c] = -INFINITY;
            before[mb][c] = -INFINITY;
            tsel[mb][c] = 0;
        }
    }
    // one fold step: scores r, r + 2 of sample block mb of node block nb of stage st.  With v1, v2 the two scores (position
    // r / 2 + 8 (nb / 2) of the class in the stage in their low four bits), the largest of {best, second, v1, v2} is
    // max3(best, v1, v2) and, because second <= best, the second largest is max(second, med3(best, v1, v2)), the maximum with two steps'
    // medians at once: nine vector instructions per four scores, plus two per stage and class for the stage number.  (The vector port is as busy as the
    // matrix pipe here: with the class's block number updated per block, two instructions more per block and class, the
    // kernel took 7 % longer.)  Four whole blocks of two bf16 parts have no register for a median that waits, and what that spills counts where a
    // tile is short: up to three stages they take each two scores' median by itself, ten instructions (search four at a time and two: 10^6 x 61 on
    // 200 nodes 128 us and 120, 10^6 x 56 on 50 77 and 71, 300,000 x 64 on 324 54 and 51, 500,000 x 64 on 400 81.5 and 82.9; fewer blocks:
    // 10^6 x 50 on 200 84 and 88, 10^6 x 12 on 600 89 and 95).
    float mid0 = 0.0f;
    auto fold_step = [&](const floatx16 (&acc)[MS], int step, int st, int nb) {
        // (a class's two steps of four scores behind one another)
        const int mb = step >> 3, p = FOUR ? (step >> 1) & 1 : step & 1, r0 = FOUR ? 4 * (2 * ((step & 7) >> 2) + (step & 1)) + p : 4 * ((step & 7) >> 1) + p, r1 = r0 + 2;
        if constexpr (CAND) {
            // A bit per score that reaches the cut, two instructions each and no branch; what a block found is noted behind
            // its last step.  (A compare and a branch per score kept the fold from running beside the MFMAs: 2.2 ns an entry at
            // K = 4096, where a tile of the search takes 1.0 ns a sample.)
            // (the set that the very first block "folds" holds the padding value, which reaches no cut)
            found[mb] = 2u * found[mb] + (acc[mb][r0] >= cut[mb] ? 1u : 0u);
            found[mb] = 2u * found[mb] + (acc[mb][r1] >= cut[mb] ? 1u : 0u);
            if (r1 == 15) {
                const unsigned long long hit = __ballot(found[mb] != 0u);
                if (hit != 0ull) {
                    const unsigned int at = queued + __builtin_amdgcn_mbcnt_hi((unsigned)(hit >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hit, 0));
                    if (found[mb] != 0u) {
                        if (at < (unsigned)QUEUE) cq.entry[at] = make_uint2(found[mb] | ((unsigned)(mb * 64 + lane) << 16), (unsigned)(st * (kNodesPerStage / 32) + nb));
                        else lost |= 1u << mb;
                    }
                    queued += (unsigned)__popcll(hit);
                    found[mb] = 0u;
                }
            }
            return;
        } else {
            const int c = 2 * (nb & 1) + p, pos = 8 * (nb >> 1);
            if (nb < 2 && r0 < 2) before[mb][c] = best[mb][c];
            const float v1 = __uint_as_float((__float_as_uint(acc[mb][r0]) & 0xfffffff0u) | (unsigned)(pos + (r0 >> 1)));
            const float v2 = __uint_as_float((__float_as_uint(acc[mb][r1]) & 0xfffffff0u) | (unsigned)(pos + (r1 >> 1)));
            const float mid = __builtin_amdgcn_fmed3f(best[mb][c], v1, v2);
            best[mb][c] = vmax3(best[mb][c], v1, v2);
            if constexpr (!FOUR) second[mb][c] = vmax(second[mb][c], mid);
            else if ((step & 1) == 0) mid0 = mid;
            else second[mb][c] = vmax3(second[mb][c], mid0, mid);
            if (nb >= 2 && r1 >= 14) tsel[mb][c] = (best[mb][c] > before[mb][c]) ? st : tsel[mb][c];
        }
    };
    // ---- stream the nodes through LDS
    const int nstages = a.kpad / kNodesPerStage;
    // what this wavefront brings in and reads is there, for all to see
    auto stage_barrier = [] {
        if constexpr (DIRECT) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else __syncthreads();
    };
    stage_barrier();

    // The scores of a node block are folded while the matrix pipe works on the next block: two sets of accumulators
    // take turns, and the fold's instructions are written between the MFMAs (the pipe is busy 32 cycles per MFMA,
    // of which the issue of the MFMA itself takes 16 on the vector port).  The very first block folds a set that
    // holds the padding value, which any real score replaces.
    floatx16 accA[MS], accB[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) accB[mb][r] = kSplitPadNorm;

    constexpr int GROUPS = HALF ? H + KB : 3 * KB + (TAIL ? 1 : 0);   // groups of MS MFMAs per node block
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int STEPS_ALL = 8 * MS;          // fold steps (two scores each) per node block
    auto block = [&](floatx16 (&cur)[MS], const floatx16 (&prev)[MS], SplitFragments<KB, FORM>& f, const char* wnext, const char* tnext, bool more,
                     int prev_st, int prev_nb) {
        if constexpr (HALF) {
            // the small products first, into accumulators that hold nothing else
#pragma unroll
            for (int grp = 0; grp < GROUPS; ++grp) {
#pragma unroll
                for (int mb = 0; mb < MS; ++mb) {
                    if (grp == 0)
                        cur[mb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(f.q[0]), fp6_operand(xq[mb][0]), zero16, 2, 2, 0, f.scales, 0, xs[mb]);
                    else if (grp < H)
                        cur[mb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(f.q[HA - 1]), fp6_operand(xq[mb][HA - 1]), cur[mb], 2, 2, 1,
                                                                                  f.scales, 1, xs[mb]);
                    else
                        cur[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.half[grp - H < 0 ? 0 : grp - H], xf[mb][grp - H < 0 ? 0 : grp - H], cur[mb], 0, 0, 0);
                    const int m = grp * MS + mb;
                    const int s0 = m * STEPS_ALL / (GROUPS * MS), s1 = (m + 1) * STEPS_ALL / (GROUPS * MS);
#pragma unroll
                    for (int sidx = s0; sidx < s1; ++sidx) fold_step(prev, sidx, prev_st, prev_nb);
                    if (mb + 1 < MS) __builtin_amdgcn_sched_barrier(0);
                }
                // LDS reads of the next block, into the registers this group has just finished with
                if (more) {
                    if (grp < H) f.read_fp6(grp, wnext, g);
                    else f.read_half(grp - H, wnext);
                    if (grp == H - 1) f.scales = *reinterpret_cast<const uint16_t*>(tnext);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        bf16x8(&wh)[KBA] = f.wh;
        bf16x8(&wl)[KBA] = f.wl;
        bf16x8& wtl = f.wtl;
        floatx16& c = f.c;
        const float4* nhnext = reinterpret_cast<const float4*>(tnext);
        // the norms of the next block replace c once the block's first group has read it
        auto next_norms = [&]() {
            if constexpr (TAIL) return;      // the norms travel inside the packed block
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 t = nhnext[2 * q];
                c[4 * q + 0] = t.x;
                c[4 * q + 1] = t.y;
                c[4 * q + 2] = t.z;
                c[4 * q + 3] = t.w;
            }
        };
        // the small products of all blocks first (lo hi, hi lo), then the large ones: what an MFMA can lose goes with what its
        // accumulator holds
#pragma unroll
        for (int grp = 0; grp < 3 * KB; ++grp) {
            const int kb = grp < 2 * KB ? grp >> 1 : grp - 2 * KB;
            const int term = grp < 2 * KB ? 1 + (grp & 1) : 0;
            const bf16x8 wa = (term == 2) ? wl[kb] : wh[kb];
#pragma unroll
            for (int mb = 0; mb < MS; ++mb) {
                cur[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa, (term == 1) ? xl[mb][kb] : xh[mb][kb],
                                                                  grp == 0 ? (TAIL ? zero16 : c) : cur[mb], 0, 0, 0);
                // this MFMA's share of the previous block's fold, fenced so that it stays behind it
                const int m = grp * MS + mb;
                const int s0 = m * STEPS_ALL / (GROUPS * MS), s1 = (m + 1) * STEPS_ALL / (GROUPS * MS);
#pragma unroll
                for (int sidx = s0; sidx < s1; ++sidx) fold_step(prev, sidx, prev_st, prev_nb);
                if (mb + 1 < MS) __builtin_amdgcn_sched_barrier(0);
            }
            // LDS reads of the next block, into the registers this group has just finished with
            if (more) {
                if (grp == 0) next_norms();
                if (term == 2) wl[kb] = *reinterpret_cast<const bf16x8*>(wnext + kb * 64 + 16);
                if (term == 0) wh[kb] = *reinterpret_cast<const bf16x8*>(wnext + kb * 64);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (TAIL) {
            constexpr int grp = 3 * KB;
#pragma unroll
            for (int mb = 0; mb < MS; ++mb) {
                cur[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wtl, xt[mb], grp == 0 ? zero16 : cur[mb], 0, 0, 0);
                const int m = grp * MS + mb;
                const int s0 = m * STEPS_ALL / (GROUPS * MS), s1 = (m + 1) * STEPS_ALL / (GROUPS * MS);
#pragma unroll
                for (int sidx = s0; sidx < s1; ++sidx) fold_step(prev, sidx, prev_st, prev_nb);
                if (mb + 1 < MS) __builtin_amdgcn_sched_barrier(0);
            }
            if (more) {
                if (grp == 0) next_norms();
                wtl = *reinterpret_cast<const bf16x8*>(wnext + KB * 64 - g * 16);    // (wnext carries g * 32)
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // CAND: direct float32 differences on the values as given over the queue's candidates, features in order
    auto serve = [&]() {
        const unsigned int n = queued < (unsigned)QUEUE ? queued : (unsigned)QUEUE;
        const int D = a.D, whole = D / 4, rest = D - 4 * whole;
        __builtin_amdgcn_wave_barrier();
        for (unsigned int e0 = 0; e0 < n; e0 += 64) {
            const uint2 e = cq.entry[e0 + lane < n ? e0 + lane : n - 1];
            unsigned int bits = e0 + lane < n ? e.x & 0xffffu : 0u;
            const unsigned int whose = e.x >> 16, smp = (whose >> 6) * 32 + (whose & 31u);
            const float* xr = a.X + (int64_t)cq.row[smp] * a.ldx;
            const unsigned int base = e.y * 32 + 4 * ((whose >> 5) & 1u);
            while (__ballot(bits != 0u) != 0ull) {
                if (bits != 0u) {
                    const int bit = 31 - __builtin_clz(bits);          // 15 - place in the order of the steps
                    bits ^= 1u << bit;
                    const int place = 15 - bit, r = FOUR ? 8 * (place >> 3) + 4 * ((place >> 1) & 1) + ((place >> 2) & 1) + 2 * (place & 1) : 4 * (place >> 2) + ((place >> 1) & 1) + 2 * (place & 1);
                    const unsigned int id = (unsigned)node_of_row((int)(base + 8 * (r >> 2) + (r & 3)), a.K);
                    if (id < (unsigned)a.K) {
                        const float* wr = a.W + (size_t)id * D;
                        float d = 0.0f;
#pragma unroll 4
                        for (int q = 0; q < whole; ++q) {
                            const float4 x4 = load4(xr + 4 * q), w4 = load4(wr + 4 * q);
                            const float d0 = x4.x - w4.x, d1 = x4.y - w4.y, d2 = x4.z - w4.z, d3 = x4.w - w4.w;
                            d = fmaf(d0, d0, d);
                            d = fmaf(d1, d1, d);
                            d = fmaf(d2, d2, d);
                            d = fmaf(d3, d3, d);
                        }
                        if (rest > 0) {          // the window [D - 4, D): its leading elements are already counted
                            const float4 x4 = load4(xr + D - 4), w4 = load4(wr + D - 4);
                            const float d1 = x4.y - w4.y, d2 = x4.z - w4.z, d3 = x4.w - w4.w;
                            if (rest > 2) d = fmaf(d1, d1, d);
                            if (rest > 1) d = fmaf(d2, d2, d);
                            d = fmaf(d3, d3, d);
                        }
                        // (no distance is negative, so their bits are in order)
                        if (d < INFINITY) atomicMin(&cq.nearest[smp], (unsigned long long)__float_as_uint(d) << 32 | id);
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        queued = 0u;
    };

    // The first node block's operands; every later block's are read while the block before it is on the matrix pipe.
    // a lane's row of a node block, and its part of what stands behind the rows: norms, or scales
    auto rows_of = [&](const char* base, int nb) { return base + (nb * 32 + j) * RS + g * (HALF ? 16 : 32); };
    auto tail_of = [&](const char* base, int nb) {
        return HALF ? base + kNodesPerStage * (RS + 4) + (nb * 32 + j) * 4 + g * 2 : base + kNodesPerStage * RS + nb * 32 * 4 + g * 16;
    };
    SplitFragments<KB, FORM> f;
    f.first(rows_of(ldsb, 0), tail_of(ldsb, 0), g);
    // One stage: the next stage travels to the idle LDS buffer from the start on (DIRECT), or global -> registers at the start and
    // registers -> the idle LDS buffer after the second block; the stage's only barrier stands in front of its last block, whose spare LDS slots then read
    // the first block of the next stage.  (With the barrier at the end of the stage a wavefront stood still for an
    // LDS write, the barrier and an LDS read once per stage; alone on its SIMD, while the unit's other workgroup
    // loads or stores its samples, that cost a fifth of its time.)  Why this is safe: a buffer's last reads, the
    // operands of its stage's last block, are issued during the block before that barrier and waited for before
    // it, so once a wavefront is past the barrier of stage s the buffer of stage s is free for stage s + 2, which
    // nobody writes before the start of stage s + 1 (DIRECT: what a wavefront has on its way it waits for in front of the same
    // barrier); and the barrier of stage s stands between every wavefront's
    // writes of stage s + 1 and the first reads of it.  That holds within a tile: a partial last stage (below) is read with no
    // barrier behind it, so who takes another tile with the same LDS puts one in between.
    constexpr int NB = kNodesPerStage / 32;
    static_assert(NB == 4, "two blocks, the LDS writes, one block, the barrier, one block");
    // A last stage that ends in whole blocks of padding nodes (K = 400: a fifth of all blocks) is left to the code behind the
    // loop, which stops at its last block of real nodes.
    const int live_last = (a.K - (nstages - 1) * kNodesPerStage + 31) / 32;
    const int nwhole = live_last < NB ? nstages - 1 : nstages;
    for (int st = 0; st < nwhole; ++st) {
        const int buf = st & 1;
        // (the last iteration reloads its own stage into the idle buffer, which keeps the loads branch-free)
        // Nine float4 per thread (D > 50) would not leave the registers for the rest: they travel in two batches.
        float4 pre0, pre1, pre2, pre3, pre4, pre5, pre6, pre7, pre8;
        static_assert(PRE <= 9, "stage copy holds at most nine float4 per thread");
        constexpr int FIRST = DIRECT ? 0 : PRE > 8 ? 5 : PRE;
        const float4* s4 = src4 + (size_t)((st + 1 < nstages) ? st + 1 : st) * STAGE_F4 + tid;
        float4* d4 = lds4 + (buf ^ 1) * (PITCH / 16) + tid;
#define SOM_PRE_LOAD(i) if constexpr (PRE > i && i < FIRST) pre##i = s4[i * kThreads];
#define SOM_PRE_STORE(i) if constexpr (PRE > i && i < FIRST) d4[i * kThreads] = pre##i;
#define SOM_PRE_LOAD2(i) if constexpr (PRE > i && i >= FIRST) pre##i = s4[i * kThreads];
#define SOM_PRE_STORE2(i) if constexpr (PRE > i && i >= FIRST) d4[i * kThreads] = pre##i;
#define SOM_PRE_ALL(op) op(0) op(1) op(2) op(3) op(4) op(5) op(6) op(7) op(8)
        if constexpr (DIRECT) {
            if (st + 1 < nstages) load_stage(st + 1, buf ^ 1);
        }
        SOM_PRE_ALL(SOM_PRE_LOAD)
        __builtin_amdgcn_sched_barrier(0);
        const char* wbuf = ldsb + (size_t)buf * PITCH;
        const char* obuf = ldsb + (size_t)(buf ^ 1) * PITCH;
        block(accA, accB, f, rows_of(wbuf, 1), tail_of(wbuf, 1), true, st - 1, 3);
        if constexpr (!DIRECT && FIRST < PRE) {
            SOM_PRE_ALL(SOM_PRE_STORE)
            SOM_PRE_ALL(SOM_PRE_LOAD2)
            __builtin_amdgcn_sched_barrier(0);
        }
        block(accB, accA, f, rows_of(wbuf, 2), tail_of(wbuf, 2), true, st, 0);
        if constexpr (DIRECT) {
        } else if constexpr (FIRST < PRE) {
            SOM_PRE_ALL(SOM_PRE_STORE2)
        } else {
            SOM_PRE_ALL(SOM_PRE_STORE)
        }
#undef SOM_PRE_LOAD
#undef SOM_PRE_STORE
#undef SOM_PRE_LOAD2
#undef SOM_PRE_STORE2
#undef SOM_PRE_ALL
        __builtin_amdgcn_sched_barrier(0);
        block(accA, accB, f, rows_of(wbuf, 3), tail_of(wbuf, 3), true, st, 1);
        stage_barrier();
        block(accB, accA, f, rows_of(obuf, 0), tail_of(obuf, 0), true, st, 2);
        if constexpr (CAND) {
            if (queued > (unsigned)QUEUE / 2) serve();
        }
    }
    // the last block's scores
    auto fold_last = [&](const floatx16 (&acc)[MS], auto nb) {
#pragma unroll
        for (int sidx = 0; sidx < STEPS_ALL; ++sidx) fold_step(acc, sidx, nstages - 1, decltype(nb)::value);
        if constexpr (!CAND) {
            // the stage number of the classes whose last block (2 of the even ones, 3 of the odd ones) did not come
#pragma unroll
            for (int mb = 0; mb < MS; ++mb)
#pragma unroll
                for (int c = 0; c < CLS; ++c)
                    if ((decltype(nb)::value < 2 && (c >> 1) <= decltype(nb)::value) || (decltype(nb)::value == 2 && (c >> 1) == 1))
                        tsel[mb][c] = (best[mb][c] > before[mb][c]) ? nstages - 1 : tsel[mb][c];
        }
    };
    if (live_last == NB) {
        fold_last(accB, std::integral_constant<int, 3>{});
    } else {
        const int st = nstages - 1;
        const char* wbuf = ldsb + (size_t)(st & 1) * PITCH;
        block(accA, accB, f, rows_of(wbuf, 1), tail_of(wbuf, 1), true, st - 1, 3);
        if (live_last == 1) {
            fold_last(accA, std::integral_constant<int, 0>{});
        } else {
            block(accB, accA, f, rows_of(wbuf, 2), tail_of(wbuf, 2), true, st, 0);
            if (live_last == 2) {
                fold_last(accB, std::integral_constant<int, 1>{});
            } else {
                block(accA, accB, f, nullptr, nullptr, false, st, 1);
                fold_last(accA, std::integral_constant<int, 2>{});
            }
        }
    }

    if constexpr (CAND) {
        // The true winner is among a sample's candidates: its score lies within the rounding bound of the best one found.  Entries
        // that lost some (the queue overflowed within a stage) or have none (no number, no cut) go to the second list, which the
        // all-nodes kernel serves.
        serve();
        lost |= (unsigned)__shfl_xor((int)lost, 32);
        const int64_t ie = wave0 + (MS > 1 ? lane : j);
        const bool writer = ie < total && (MS > 1 || g == 0);
        const unsigned long long best_key = cq.nearest[MS > 1 ? lane : j];
        const bool served = best_key != ~0ull && ((lost >> (MS > 1 ? g : 0)) & 1u) == 0u;
        const int64_t i = writer ? (int64_t)a.recheck[ie] : 0;
        if (writer && served) a.bmu[i] = (int32_t)(unsigned)best_key;
        list_push(&a.scal[a.slot2], a.recheck2, nullptr, writer && !served, i, 0.0f);
        return;
    }
    // ---- winners and bounds
    const float wmax2 = __uint_as_float(a.norms[0]);
    const float wmax = sqrtf(wmax2) * 1.000001f;
    // |w|^2 / 2 in the accumulators: see (2) at the start of the tile; and six units as for the products
    constexpr float kErrNorm = ((TAIL || HALF ? 16.256f : 48.768f * KB) + 6.0f) * 5.9604645e-08f;
    // (square roots here are the hardware's, good to a unit in the last place; the factors behind them cover it)
    auto root = [](float v) { return __builtin_amdgcn_sqrtf(v); };
    // Lane (j, g) finishes sample j of block g (MS = 1: half 0 does): the halves trade what they hold of each other's block, and
    // all eight class winners of a sample meet in one lane: places 0 to 3 from half 0's rows, 4 to 7 from half 1's.
    static_assert(MS <= 2, "a block per lane half");
    float won[8], most;
    int from[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        won[c] = best[0][c];
        won[4 + c] = best[MS - 1][c];
        swap_halves(won[c], won[4 + c]);
        from[c] = tsel[0][c];
        from[4 + c] = tsel[MS - 1][c];
        swap_halves(from[c], from[4 + c]);
    }
    {
        float m0 = fmaxf(fmaxf(second[0][0], second[0][1]), fmaxf(second[0][2], second[0][3]));
        float m1 = fmaxf(fmaxf(second[MS - 1][0], second[MS - 1][1]), fmaxf(second[MS - 1][2], second[MS - 1][3]));
        swap_halves(m0, m1);
        most = fmaxf(m0, m1);
    }
    // HALF: the scores stay at the scale they were formed at, and bounds and cuts go there: taken to the values' own, a score of zero
    // or one that is subnormal there would lose its position.
    const int up = HALF ? __float_as_int(stash[5 * kThreads]) : 0;
    // winner and runner-up (equal scores are a near tie, decided elsewhere: any of them)
    float r_best = won[0], r_second = -INFINITY;
#pragma unroll
    for (int q = 1; q < 7; q += 2) {
        const float mid = __builtin_amdgcn_fmed3f(r_best, won[q], won[q + 1]);
        r_best = fmaxf(fmaxf(r_best, won[q]), won[q + 1]);
        r_second = fmaxf(r_second, mid);
    }
    r_second = fmaxf(fmaxf(r_second, fminf(r_best, won[7])), most);
    r_best = fmaxf(r_best, won[7]);
    // row of a score that won place q in stage st
    auto row_of = [](float v, int st, int q) {
        const unsigned pos = __float_as_uint(v) & 15u;
        return st * kNodesPerStage + (int)(((pos & 8u) << 3) + ((pos & 6u) << 2) + ((pos & 1u) << 1)) + 32 * ((q >> 1) & 1) + (q & 1) + 4 * (q >> 2);
    };
    int r_stage = from[0], r_place = 0;
#pragma unroll
    for (int q = 1; q < 8; ++q) {
        r_stage = won[q] == r_best ? from[q] : r_stage;
        r_place = won[q] == r_best ? 32 * ((q >> 1) & 1) + (q & 1) + 4 * (q >> 2) : r_place;
    }
    int r_row = row_of(r_best, r_stage, 0) + r_place;
    r_row = (r_row >= 0 && r_row < a.K) ? r_row : a.K - 1;               // (only padding or non-finite scores get here)
    const int64_t i = wave0 + (MS > 1 ? lane : j);
    const bool r_valid = i < a.m && (MS > 1 || g == 0);
    // the winner's squared norm from the stage blob, and the sample's figures from the start of the tile
    const char* blob = reinterpret_cast<const char*>(a.stage16) + (size_t)(r_row / kNodesPerStage) * STAGE_F4 * 16;
    const float wn = -2.0f * reinterpret_cast<const float*>(blob + (size_t)kNodesPerStage * RS)[r_row % kNodesPerStage];
    // The winner's score errs by its own norm's bound, which bounds its distance (far).  A node that is in truth as near as the winner
    // lies within that distance of the sample, so its norm is at most |x| + far (and at most the largest), and it lies within 2 far of the
    // winner; no other node can spoil the decision.  The position bits change a score by at most 2^-19 of itself, and a rival's
    // score is within the bound of the best one.
    const float nx = stash[0], wb = fminf(root(wn + (HALF ? kSquaresFloor : 0.0f)) * 1.0001f, wmax);
    const float top = HALF ? ldexpf(r_best, -up) : r_best;
    const float bits = fabsf(top) * (1.01f * 3.8146973e-06f);
    float bound;
    if constexpr (HALF) {
        const float err_w = stash[kThreads], nr = stash[2 * kThreads], nl = stash[3 * kThreads], qh = stash[4 * kThreads];
        static_assert(25 - kHalfNorm + kHalfThird == 21, "5.0e-7: 2^-21");
        const float back_w = power_of_two(-sw), err_n = back_w * back_w * 5.0e-7f + kSquaresFloor;
        // what a score errs by for each unit of its node's second part, of what fp6 leaves of its first, and of its second part
        constexpr float small = 80.0f * (H + 2) * 5.9604645e-08f;
        const float by_lo = nr + qh + nl + nx * small, by_qh = nl + nr, by_ql = nl + qh;
        // those of a node of this norm, in the order of norms[1..3] and norms[4..6]
        auto over = [&](int part, float norm) {
            return fminf(__uint_as_float(a.norms[1 + part]) * (norm + kHalfNearest * back_w), __uint_as_float(a.norms[4 + part])) * 1.001f;
        };
        const float lo_b = over(0, wb), qh_b = over(1, wb), ql_b = over(2, wb);
        const float err_b = (err_w + nr) * wb + by_lo * lo_b + by_qh * qh_b + (by_ql + nx + wb) * ql_b + err_n + 0.5f * kErrNorm * wb * wb;
        const float far = root(fmaxf(nx * nx * 1.00001f - 2.0f * top, 0.0f) * 1.00001f + 2.0f * (err_b + bits)) * 1.0001f;
        const float reach = (nx + far) * 1.0001f, wo = fminf(reach, wmax), two = wb + wo;
        bound = ldexpf(err_w * two + by_lo * (lo_b + over(0, wo)) + by_qh * (qh_b + over(1, wo)) + (by_ql + far) * (ql_b + over(2, wo)) +
                           nr * fminf(2.0f * far, two) + 2.0f * err_n + 0.5f * kErrNorm * (wb * wb + wo * wo) + bits,
                       up);
        if (!(reach < __uint_as_float(0x7f800000u - a.norms[7]))) bound = INFINITY;          // (a node without a row may be as near)
    } else {
        const float err_0 = stash[kThreads];
        const unsigned int two = __float_as_uint(stash[2 * kThreads]);
        const float err_w = __uint_as_float(two & 0xffff0000u), nr = __uint_as_float(two << 16);
        const float rest_w = root(__uint_as_float(a.norms[2]) + kSquaresFloor) * 1.0079f;
        const float err_b = (err_w + nr) * wb + err_0 + (nx + wb) * rest_w + 0.5f * kErrNorm * wb * wb;
        const float far2 = fmaxf(nx * nx * 1.00001f - 2.0f * r_best, 0.0f) * 1.00001f + 2.0f * (err_b + bits);
        const float far = root(far2) * 1.0001f;
        const float wo = fminf((nx + far) * 1.0001f, wmax);
        bound = err_w * (wb + wo) + 2.0f * err_0 + nr * fminf(2.0f * far, wb + wo) + 2.0f * far * rest_w + 0.5f * kErrNorm * (wb * wb + wo * wo) + bits;
    }
    const bool close = r_valid && a.K > 1 && !((r_best - r_second) > bound);
    // Candidates: the class winners that reach the cut, four at most on small maps; complete when no class's runner-up reaches it.
    // Otherwise (or with 16-bit ids not enough) the sample goes on the list of the candidate pass.
    const float cut_at = r_best - bound;
    bool open = !(most < cut_at) || a.K > kPairNodes;
    if (__ballot(close) != 0ull) {
        unsigned int p0 = 0xffffffffu, p1 = 0xffffffffu, p2 = 0xffffffffu, p3 = 0xffffffffu;      // eight places, the used ones in front
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const bool hit = won[q] >= cut_at;
            const unsigned id = (unsigned)row_of(won[q], from[q], q);
            p3 = hit ? (p3 << 16) | (p2 >> 16) : p3;
            p2 = hit ? (p2 << 16) | (p1 >> 16) : p2;
            p1 = hit ? (p1 << 16) | (p0 >> 16) : p1;
            p0 = hit ? (p0 << 16) | id : p0;
        }
        open = open || (p2 != 0xffffffffu && a.K < kPairMany);
        if (close && !open) {
            if (a.K >= kPairMany) *reinterpret_cast<uint4*>(a.pairs + 4 * i) = make_uint4(p0, p1, p2, p3);
            else *reinterpret_cast<uint2*>(a.pairs + 2 * i) = make_uint2(p0, p1);
        }
    }
    int near = 0;
    if (r_valid) {
        if (a.qe) {
            // The statistic n_recheck counts the near ties: best two scores inside a band of fixed relative width, which takes 3 * 2^-18
            // for the cut (four times less than it can lose: a figure to compare runs by, not a bound) and all MFMAs at the full
            // magnitude.  Only those that this sample's own bound leaves open are listed.
            // (the MFMAs of two bf16 parts: three a 16-feature block, one for a remainder of up to four features)
            const int left = a.D % 16, mfmas = left >= 1 && left <= 4 ? 49 * (a.D / 16) + 17 : 49 * ((a.D + 15) / 16);
            const float rel = 2.0f * (3.0f * 3.8146973e-06f * 1.0078125f + (float)(mfmas + 1) * 5.9604645e-08f + 1.9073486e-06f) + 12.0f * 5.9604645e-08f;
            const float band = 0.5f * rel * ((nx * wb + 0.5f * wb * wb) + (nx * wmax + 0.5f * wmax2));
            near = (close || (a.K > 1 && !((r_best - r_second) > (HALF ? ldexpf(band, up) : band)))) ? 1 : 0;
        }
        a.bmu[i] = node_of_row(r_row, a.K);
        a.cut_all[i] = !close ? kNotListed : open ? list_cut(cut_at) : kPairs;
    }
    if (a.qe) group_qe_add(a.qe_part, 0.0, 0.0, near);
}

// full tiles for the workgroups below a.full_tiles, half tiles for the last partial round (as bmu_kernel)
template <int KB, int FORM, int MS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_split_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    if ((int64_t)blockIdx.x < a.full_tiles) {
        bmu_split_tile<KB, FORM, MS, false>(a, 0, blockIdx.x, 0u, lds4);
    } else if constexpr (MS > 1) {
        constexpr int64_t per_full = (int64_t)kWavesPerGroup * MS * 32;
        bmu_split_tile<KB, FORM, MS / 2, false>(a, a.full_tiles * per_full, (int64_t)blockIdx.x - a.full_tiles, 0u, lds4);
    }
}

// candidate pass of the split search: a fixed grid walks the tiles of the list.  Whole rounds of two tiles per compute unit,
// and what is left (a short list: everything) in tiles of half the size: a list of 1032 tiles took three rounds for two.
template <int KB, int FORM, int MS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_split_cand_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    const unsigned int count = a.scal[a.slot];
    if (!cand_pass_serves(a, count)) return;
    constexpr unsigned int per_tile = (unsigned int)kWavesPerGroup * MS * 32;
    static_assert(MS == 2, "half tiles");
    constexpr unsigned int round = 512;
    const unsigned int full = count <= kCandHalfTiles ? 0u : count / per_tile / round * round;
    const unsigned int halves = (count - full * per_tile + per_tile / 2 - 1) / (per_tile / 2);
    for (unsigned int t = blockIdx.x; t < full + halves; t += gridDim.x) {
        BmuArgs b = a;                     // (nothing derived from these is carried from tile to tile: registers)
        asm volatile("" : "+s"(b.centre), "+s"(b.D), "+s"(b.tail_r), "+s"(b.K));
        if (t < full) bmu_split_tile<KB, FORM, MS, true>(b, 0, t, count, lds4);
        else bmu_split_tile<KB, FORM, MS / 2, true>(b, (int64_t)full * per_tile, t - full, count, lds4);
        // The next tile starts by filling buffer 0, and a tile's last stage, where it is a partial one, is read behind the tile's
        // last barrier: from buffer 0 with an odd number of stages.  (A wavefront there may be far behind the others: it may have
        // had its queue to serve.)
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------------
// the same search for D > 64: features go through in chunks of 50, 56 or 64.  A wavefront owns one block of 32
// samples; the accumulators of a stage's four node blocks stay live across the chunks, the samples' features of
// the current chunk are re-read from memory once per stage (one workgroup touches 128 rows).
// ---------------------------------------------------------------------------------------------------------
// CAND as in bmu_tile: the candidate pass over the first `count` entries of the re-decision list.
template <int STEPS, bool CAND>
__device__ __forceinline__ void bmu_wide_tile(const BmuArgs& a, int64_t tile_index, unsigned int count, float4* lds4)
{
    constexpr int CH = 2 * STEPS;                        // features per chunk
    constexpr int STRIDE = 2 * STEPS + 1, NBS = kNodesPerStage / 32;
    constexpr int STAGE_FLOATS = stage_floats_for(STRIDE);
    constexpr int STAGE_F4 = STAGE_FLOATS / 4;
    constexpr int PRE = STAGE_F4 / kThreads;
    static_assert(PRE <= 9, "stage copy holds at most nine float4 per thread");
    float* lds = reinterpret_cast<float*>(lds4);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int j = lane & 31, g = lane >> 5;
    const int64_t i = (tile_index * kWavesPerGroup + wave) * 32 + j;      // sample position, or list entry (CAND)
    const int64_t total = CAND ? (int64_t)count : a.m;
    const bool valid = i < total;
    int64_t ii = valid ? i : total - 1;
    float cut = NAN;                                                        // CAND; no score compares >= NaN
    CandSet noted;
    if constexpr (CAND) {
        if (valid) cut = a.cutv[ii];
        ii = (int64_t)a.recheck[ii];
    }
    const int64_t row = a.idx ? (int64_t)a.idx[ii] : ii;
    const float* xr = a.X + row * a.ldx;

    float best = -INFINITY, second = -INFINITY;
    int rsel = 0, tsel = 0;
    const int nstages = a.kpad / kNodesPerStage;
    const int nch = (a.D + CH - 1) / CH;
    const int nq = nstages * nch;
    const float4* src4 = reinterpret_cast<const float4*>(a.stage);
    {
        float4 first[PRE];
#pragma unroll
        for (int p = 0; p < PRE; ++p) first[p] = src4[tid + p * kThreads];
#pragma unroll
        for (int p = 0; p < PRE; ++p) lds4[tid + p * kThreads] = first[p];
    }
    __syncthreads();

    floatx16 acc[NBS];
    int st = 0, ch = 0;
    // Centred features of the current chunk.  Lane (j, g) holds STEPS contiguous features of the chunk, the window the weight preparation laid the stage
    // columns out for: [CH ch + STEPS g, + STEPS), moved back to [D - STEPS, D) where it would pass the end of the
    // row.  Every chunk therefore comes in as STEPS / 4 16-byte loads per lane (4-byte aligned addresses are
    // enough for them; STEPS = 25 adds one dword), with no bounds to check and nothing read outside the row.
    auto window_of = [&](int chunk) {
        const int first = CH * chunk + STEPS * g;
        return first < a.D - STEPS ? first : a.D - STEPS;
    };
    float x[STEPS];
    {
        const float* xc = xr + window_of(0);
        const float* cc = a.centre + window_of(0);
#pragma unroll
        for (int t = 0; t < STEPS / 4; ++t) {
            const float4 v = load4(xc + 4 * t), c = load4(cc + 4 * t);
            x[4 * t + 0] = v.x - c.x;
            x[4 * t + 1] = v.y - c.y;
            x[4 * t + 2] = v.z - c.z;
            x[4 * t + 3] = v.w - c.w;
        }
#pragma unroll
        for (int s = STEPS / 4 * 4; s < STEPS; ++s) x[s] = xc[s] - cc[s];
    }
    for (int q = 0; q < nq; ++q) {
        const int buf = q & 1;
        float4 pre0, pre1, pre2, pre3, pre4, pre5, pre6, pre7, pre8;
        {
            const int nxt = (q + 1 < nq) ? q + 1 : q;
            const float4* s4 = src4 + (size_t)nxt * STAGE_F4 + tid;
#define SOM_PRE_LOAD(i) if constexpr (PRE > i) pre##i = s4[i * kThreads];
            SOM_PRE_LOAD(0) SOM_PRE_LOAD(1) SOM_PRE_LOAD(2) SOM_PRE_LOAD(3) SOM_PRE_LOAD(4)
            SOM_PRE_LOAD(5) SOM_PRE_LOAD(6) SOM_PRE_LOAD(7) SOM_PRE_LOAD(8)
#undef SOM_PRE_LOAD
        }
        // the samples' next chunk travels to registers during this chunk's arithmetic, like the next stage blob
        // (and with them the matching entries of the centre vector: vector loads cost no matrix-pipe time, a
        // select between two scalar values per entry would)
        float xn[STEPS], cn[STEPS];
        {
            const int chn = (ch + 1 == nch) ? 0 : ch + 1;
            const int w0 = window_of(chn);
            const float* cc = a.centre + w0;
            const float* xc = xr + w0;
#pragma unroll
            for (int t = 0; t < STEPS / 4; ++t) {
                const float4 c = load4(cc + 4 * t);
                cn[4 * t + 0] = c.x;
                cn[4 * t + 1] = c.y;
                cn[4 * t + 2] = c.z;
                cn[4 * t + 3] = c.w;
                const float4 v = load4(xc + 4 * t);
                xn[4 * t + 0] = v.x;
                xn[4 * t + 1] = v.y;
                xn[4 * t + 2] = v.z;
                xn[4 * t + 3] = v.w;
            }
#pragma unroll
            for (int s = STEPS / 4 * 4; s < STEPS; ++s) {
                cn[s] = cc[s];
                xn[s] = xc[s];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const float* wbuf = lds + buf * STAGE_FLOATS;
        const float* nbuf = wbuf + kNodesPerStage * STRIDE;
        // As in bmu_kernel the LDS reads of node block nb + 1 are written into the MFMA sequence of block nb (one
        // read per MFMA) where the registers allow it (STEPS <= 28); only the first block of a chunk waits for LDS.
        constexpr bool PIPE = STEPS <= 28;
        float wa[PIPE ? STEPS : 1];
        if constexpr (PIPE) {
            const float* wrow = wbuf + j * STRIDE + g;
#pragma unroll
            for (int s = 0; s < STEPS; ++s) wa[s] = wrow[2 * s];
        }
#pragma unroll
        for (int nb = 0; nb < NBS; ++nb) {
            if (ch == 0) {
                const float4* nh = reinterpret_cast<const float4*>(nbuf + nb * 32 + 4 * g);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float4 v = nh[2 * t];
                    acc[nb][4 * t + 0] = v.x;
                    acc[nb][4 * t + 1] = v.y;
                    acc[nb][4 * t + 2] = v.z;
                    acc[nb][4 * t + 3] = v.w;
                }
            }
            // The chunk's 64-feature partial product is summed on its own, from zero, and then added to the
            // running score: every rounding inside the chunk is relative to the chunk's own magnitude
            // |x_chunk| |w_chunk|, and those add up to at most |x| |w| over the chunks (Cauchy-Schwarz), so the
            // error bound grows with 2 STEPS + nch roundings per score instead of 2 STEPS nch.
            const float* wrow = wbuf + (nb * 32 + j) * STRIDE + g;
            floatx16 part;
#pragma unroll
            for (int r = 0; r < 16; ++r) part[r] = 0.0f;
            if constexpr (PIPE) {
                const float* wnext = wrow + 32 * STRIDE;
                float wn[STEPS];
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    part = __builtin_amdgcn_mfma_f32_32x32x2f32(wa[s], x[s], part, 0, 0, 0);
                    if (nb + 1 < NBS) {
                        wn[s] = wnext[2 * s];
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // one LDS read
                    }
                }
                if (nb + 1 < NBS) {
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) wa[s] = wn[s];
                }
            } else {
#pragma unroll
                for (int s = 0; s < STEPS; ++s)
                    part = __builtin_amdgcn_mfma_f32_32x32x2f32(wrow[2 * s], x[s], part, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[nb][r] += part[r];
            if (CAND && ch == nch - 1) {
                const int tile = st * NBS + nb;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (acc[nb][r] >= cut) noted.note(tile * 32 + 4 * g, 8 * (r >> 2) + (r & 3));
            }
            if (!CAND && ch == nch - 1) {
                const int tile = st * NBS + nb;
                const float before = best;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float v = acc[nb][r];
                    rsel = (v > best) ? r : rsel;
                    second = __builtin_amdgcn_fmed3f(best, second, v);
                    best = vmax(best, v);
                }
                tsel = (best > before) ? tile : tsel;
            }
        }
        {
            float4* d4 = lds4 + (buf ^ 1) * STAGE_F4 + tid;
#define SOM_PRE_STORE(i) if constexpr (PRE > i) d4[i * kThreads] = pre##i;
            SOM_PRE_STORE(0) SOM_PRE_STORE(1) SOM_PRE_STORE(2) SOM_PRE_STORE(3) SOM_PRE_STORE(4)
            SOM_PRE_STORE(5) SOM_PRE_STORE(6) SOM_PRE_STORE(7) SOM_PRE_STORE(8)
#undef SOM_PRE_STORE
        }
        __syncthreads();
        if (++ch == nch) {
            ch = 0;
            ++st;
        }
#pragma unroll
        for (int s = 0; s < STEPS; ++s) x[s] = xn[s] - cn[s];
    }

    if constexpr (CAND) {
        if (valid) a.cand[(size_t)i * 2 + g] = noted.packed();
        return;
    }
    // ---- join the two half-wavefronts; squared norm and exact winner distance from memory, half the features each
    int node = tsel * 32 + 8 * (rsel >> 2) + 4 * g + (rsel & 3);
    const float ob = __shfl_xor(best, 32), os = __shfl_xor(second, 32);
    const int on = __shfl_xor(node, 32);
    const float sec = fmaxf(fmaxf(second, os), fminf(best, ob));
    const bool other = (ob > best) || (ob == best && on < node);
    const float bst = other ? ob : best;
    node = other ? on : node;
    node = node < a.K ? node : a.K - 1;
    float xn = 0.f, part = 0.f;
    const float* wr = a.W + (size_t)node * a.D;
    for (int f = g; f < a.D; f += 2) {
        const float xv = xr[f];
        const float xc = xv - a.centre[f];
        const float df = xv - wr[f];
        xn = fmaf(xc, xc, xn);
        part = fmaf(df, df, part);
    }
    xn += __shfl_xor(xn, 32);
    part += __shfl_xor(part, 32);
    double qs = 0.0, qs2 = 0.0;
    const float wmax2 = __uint_as_float(a.scal[0]);
    const float wmax = sqrtf(wmax2) * 1.000001f;
    // per score: 2 STEPS roundings inside the chunks (see the stage loop), nch chunk additions, one for
    // -|w|^2/2; two scores, plus the centring roundings and slack as in bmu_kernel
    const float rel = (float)(4 * STEPS + 2 * nch + 12) * 5.9604645e-08f;
    const float bound = (sqrtf(xn) * wmax + 0.5f * wmax2) * rel;
    const bool mine = valid && g == 0;
    const bool close = mine && a.K > 1 && !((bst - sec) > bound);
    if (mine) {
        a.bmu[i] = node;
        if (a.d2) a.d2[i] = part;
        if (!close) {
            qs = sqrt((double)part);
            qs2 = (double)part;
        }
    }
    if (mine) a.cut_all[i] = close ? list_cut(bst - bound) : kNotListed;
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

template <int STEPS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_wide_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    bmu_wide_tile<STEPS, false>(a, blockIdx.x, 0u, lds4);
}

template <int STEPS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_wide_cand_kernel(const BmuArgs a)
{
    extern __shared__ float4 lds4[];
    const unsigned int count = a.scal[a.slot];
    if (!cand_pass_serves(a, count)) return;
    constexpr int64_t per_tile = (int64_t)kWavesPerGroup * 32;
    for (int64_t t = blockIdx.x; t * per_tile < (int64_t)count; t += gridDim.x) bmu_wide_tile<STEPS, true>(a, t, count, lds4);
}

// ---------------------------------------------------------------------------------------------------------
// exact re-decision of the listed samples by direct differences, sum_d (x_d - w_kd)^2 for every node.
// A workgroup takes kExactGroup samples at a time; thread t owns nodes t, t + 256, ... so one coalesced read of
// the transposed weights serves all samples of the group, and the samples' features are broadcast from LDS.
// The inner loop is one v_sub and one v_fmac per (sample, node, feature) with nothing else in the way, i.e. the
// plain vector-ALU rate: 2 K D lane-operations per sample (2.6 ns at K = 1024, D = 50 on 256 compute units; 3.8 ns
// measured with every sample listed).  Larger groups or prefetched weights were measured and change nothing.
// ---------------------------------------------------------------------------------------------------------
constexpr int kExactGroup = 8;
constexpr int kExactNodesPerThread = 2;
constexpr size_t kExactLds = 64 * (kExactGroup / 4) * 16;      // bytes: a slab of 64 features of the samples in hand
constexpr int kExactThreads = 512;         // K = 1024 in one sweep; 256 threads of four nodes each took 25 us for any short list (a chain
                                           // of thirteen batches of loads with little to hide them), these take 14

// ---------------------------------------------------------------------------------------------------------
// Direct differences over the nodes the candidate pass noted (the true winner is among them: its score lies
// within the rounding bound of the best one found).  Sixteen lanes per list entry, each a sixteenth of the
// features; lowest distance, then lowest node index.  Entries whose slots overflowed (more than seven candidates
// in one half) or that noted nothing (non-finite scores) go to the second list, which the all-nodes kernel serves.
// ---------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) bmu_cand_exact_kernel(const BmuArgs a)
{
    const unsigned int count = a.scal[a.slot];
    if (!cand_pass_serves(a, count)) return;
    const int sub = threadIdx.x & 15;
    constexpr unsigned int per_group = 256 / 16;
    constexpr int kMost = 2 * (kCandSlots - 1);        // candidates of one sample at most
    double qs = 0.0, qs2 = 0.0;
    for (unsigned int p0 = blockIdx.x * per_group; p0 < count; p0 += gridDim.x * per_group) {
        const unsigned int p = p0 + (threadIdx.x >> 4);
        const bool live = p < count;
        const unsigned int pc = live ? p : count - 1;
        const int64_t i = (int64_t)a.recheck[pc];
        const ulonglong2 h0 = a.cand[(size_t)pc * 2], h1 = a.cand[(size_t)pc * 2 + 1];
        const int64_t row = a.idx ? (int64_t)a.idx[i] : i;
        const float* xr = a.X + row * a.ldx;
        const int c0 = cand_count(h0), c1 = cand_count(h1);
        bool served = c0 < kCandSlots && c1 < kCandSlots && c0 + c1 > 0;
        const int c = served ? c0 + c1 : 0;
        // Both halves' candidates form one dense list of c places, taken four at a time (most samples have no more):
        // the loads of a batch (four rows of W, a quarter of 64 features per lane) are issued together, and batches
        // nobody in the wavefront needs are skipped.
        float bd = INFINITY;
        int bk = 0x7fffffff;
        constexpr int kBatch = 4;
        for (int t0 = 0; t0 < kMost; t0 += kBatch) {
            if (__ballot(c > t0) == 0ull) break;
            int node[kBatch];
            float d[kBatch];
#pragma unroll
            for (int tt = 0; tt < kBatch; ++tt) {
                const int t = t0 + tt, u = t - c0;
                const int k = (t < c0) ? cand_id(h0, t < kCandSlots - 1 ? t : 0)
                                       : cand_id(h1, u < kCandSlots - 1 ? u : 0);
                node[tt] = (t < c && k < a.K) ? k : -1;
                d[tt] = 0.0f;
            }
            for (int f0 = 0; f0 < a.D; f0 += 64) {
                float xv[4], wv[kBatch][4];
                int fo[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int f = f0 + 16 * q + sub;
                    fo[q] = f < a.D ? f : -1;
                    xv[q] = xr[fo[q] >= 0 ? f : a.D - 1];
                }
#pragma unroll
                for (int tt = 0; tt < kBatch; ++tt) {
                    const float* wr = a.W + (size_t)(node[tt] >= 0 ? node[tt] : 0) * a.D;
#pragma unroll
                    for (int q = 0; q < 4; ++q) wv[tt][q] = wr[fo[q] >= 0 ? fo[q] : a.D - 1];
                }
#pragma unroll
                for (int tt = 0; tt < kBatch; ++tt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float df = fo[q] >= 0 ? xv[q] - wv[tt][q] : 0.0f;
                        d[tt] = fmaf(df, df, d[tt]);
                    }
            }
#pragma unroll
            for (int tt = 0; tt < kBatch; ++tt) {
                float v = d[tt];
                v += __shfl_xor(v, 8);
                v += __shfl_xor(v, 4);
                v += __shfl_xor(v, 2);
                v += __shfl_xor(v, 1);
                const int k = node[tt];
                if (k >= 0 && (v < bd || (v == bd && k < bk))) {
                    bd = v;
                    bk = k;
                }
            }
        }
        served = served && bk < a.K;
        const bool mine = live && sub == 0;
        if (mine && served) {
            a.bmu[i] = bk;
            if (a.d2) a.d2[i] = bd;
            qs += sqrt((double)bd);
            qs2 += (double)bd;
        }
        list_push(&a.scal[a.slot2], a.recheck2, nullptr, mine && !served, i, 0.0f);
    }
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

// ---------------------------------------------------------------------------------------------------------
// The pair list: samples whose candidates (at most eight) the split search already knows (D <= 64).
// A wavefront takes a round of sixteen entries at a time, on its own (no barrier): LP lanes (4, 8 or 16, sixteen bytes of a row each) fetch
// an entry's rows, the sample's and two candidates', in coalesced loads; the differences meet in the wavefront's part of LDS, the next entries'
// rows are requested, and one lane per candidate adds the squares up, features in order as the other re-decisions do;
// lowest distance, then lowest node index.
// The chain sample position -> ids and row number -> rows is three dependent trips to memory: positions are read three rounds ahead, ids and
// row numbers two, rows one, each by one lane an entry, and two workgroups of eight wavefronts fit a unit.
// What bounds it beside the rows' lines is instructions: a lane of the sum is a whole wavefront's instruction for 32 candidates at most, so
// the differences are formed where all lanes have a share of them, and sixteen entries share the sum.  (Eight entries a round, three rows of
// each in LDS: 10^7 x 50 on a tree's 1024 nodes, half of the rows listed, 636 us, 529 this way; 10^6 x 50 on 4096 nodes 76 and 58.)
// Sums across the LP lanes would take fewer still, but they add in another order, and a sample that lies between two nodes
// must not go to one of them in a look-up and to the other in an epoch.
// The few entries with a third to an eighth candidate wait in LDS until there is a round of them, two candidates at a time, which then takes
// its turn among the others: its rows, too, are on their way during the round before.  (Served between two rounds, with the next one's rows
// fetched again behind them: 529 us, 483 this way; 10^6 x 50 on 4096 nodes 58 and 52.)
// ---------------------------------------------------------------------------------------------------------
constexpr int pair_lanes(int D) { return D <= 16 ? 4 : D <= 32 ? 8 : 16; }
constexpr int kPairRound = 16;                                          // entries of a round
// float4 of LDS that a wavefront's entries take: two differences (an odd number each, so that the lanes' 16-byte reads fall into distinct
// banks), what two rounds and twice as many waiting entries note, and their row numbers
__host__ __device__ constexpr int pair_lds_f4(int D) { return kPairRound * (2 * (((D + 3) / 4) | 1) + 2 + 2 + 1); }

template <int LP>
__device__ __forceinline__ void pair_list(const BmuArgs& a, float4* __restrict__ lds)
{
    constexpr int ROUND = kPairRound, GROUPS = 64 / LP, EACH = ROUND / GROUPS;
    static_assert(2 * ROUND <= 64, "a lane a candidate");
    const unsigned int count = a.scal[a.slot + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = lane & (LP - 1), grp = lane / LP;
    const int D = a.D, whole = D / 4, rest = D - 4 * whole;
    const int stride = ((D + 3) / 4) | 1;             // float4 of a difference
    float4* const rows = lds + wave * pair_lds_f4(D);
    // What a round's entries note, [round's parity][entry]: of new ones two words of ids and the sample's position; of entries that waited
    // the next two ids, the position, the nearest so far (distance; row of the stages, and which word of its ids the two are).
    uint4* const info = reinterpret_cast<uint4*>(rows + ROUND * 2 * stride);
    uint4* const later = info + 2 * ROUND;                          // [2 ROUND]
    uint32_t* const info_row = reinterpret_cast<uint32_t*>(later + 2 * ROUND);    // [2][ROUND], the samples' rows
    uint32_t* const later_row = info_row + 2 * ROUND;               // [2 ROUND]
    constexpr unsigned int kNoRow = 0xffffffu;
    const int pair_shift = a.K >= kPairMany ? 2 : 1;                // words of an entry's ids
    unsigned int waiting = 0u;
    const int start = 4 * sub < D - 4 ? 4 * sub : D - 4;           // window inside the row
    const bool own = 4 * sub < D;
    const unsigned int step = gridDim.x * (kExactThreads / 64) * ROUND;
    const unsigned int first = (blockIdx.x * (kExactThreads / 64) + wave) * ROUND;
    if (first >= count) return;
    const unsigned int k_most = (unsigned int)a.K - 1u;
    const char* const wrow = reinterpret_cast<const char*>(a.wrow);
    // (a map of 65535 nodes x 64 features has 16 MB)
    auto row_of = [&](unsigned int id) {
        return load4(reinterpret_cast<const float*>(wrow + (((id < k_most ? id : k_most) * (unsigned)D + (unsigned)start) * 4u)));
    };
    float4 x[EACH], w[EACH][2];
    // entry u's rows for this lane's window (a single candidate's twice)
    auto fetch = [&](int u, unsigned int both, uint32_t row) {
        const unsigned int i0 = both & 0xffffu, i1 = both >> 16;
        x[u] = load4(a.X + (int64_t)row * a.ldx + start);
        w[u][0] = row_of(i0);
        w[u][1] = row_of(i1 == 0xffffu ? i0 : i1);
    };
    auto lay = [&](int u) {
        float4* r = rows + (GROUPS * u + grp) * 2 * stride + sub;
        if (own) {
#pragma unroll
            for (int c = 0; c < 2; ++c)
                r[c * stride] = make_float4(x[u].x - w[u][c].x, x[u].y - w[u][c].y, x[u].z - w[u][c].z, x[u].w - w[u][c].w);
        }
    };
    // this lane's candidate: entry lane / 2, place lane % 2
    const int e = (lane >> 1) & (ROUND - 1), c = lane & 1;
    float bd;
    int bk;                                           // row of the stages
    // (which node a row holds matters only where two are exactly as near)
    auto nearer = [&](float d, int k) {
        bool take = d < bd;
        const bool tie = d == bd && d < INFINITY;
        if (__ballot(tie) != 0ull) take = take || (tie && node_of_row(k, a.K) < node_of_row(bk, a.K));
        bd = take ? d : bd;
        bk = take ? k : bk;
    };
    auto sum = [&](unsigned int both) {
        const unsigned int id = c == 0 ? both & 0xffffu : both >> 16;
        const float4* r = rows + (2 * e + c) * stride;
        float d = 0.0f;
        if (lane < 2 * ROUND) {
#pragma unroll 4
            for (int q = 0; q < whole; ++q) {
                const float4 v = r[q];
                d = fmaf(v.x, v.x, d);
                d = fmaf(v.y, v.y, d);
                d = fmaf(v.z, v.z, d);
                d = fmaf(v.w, v.w, d);
            }
            if (rest > 0) {          // the window [D - 4, D): its leading elements are already counted
                const float4 v = r[whole];
                if (rest > 2) d = fmaf(v.y, v.y, d);
                if (rest > 1) d = fmaf(v.z, v.z, d);
                d = fmaf(v.w, v.w, d);
            }
        }
        nearer(id != 0xffffu ? d : INFINITY, (int)id);
        nearer(__shfl_xor(bd, 1), __shfl_xor(bk, 1));
    };
    // entry `lane % ROUND` of the round at p (behind the list's end its last one)
    auto position = [&](unsigned int p) {
        const unsigned int q = p + (lane & (ROUND - 1));
        return a.recheck_end[-1 - (int64_t)(q < count ? q : count - 1)];
    };
    auto ids_of = [&](uint32_t at) { return *reinterpret_cast<const uint2*>(a.pairs + ((int64_t)at << pair_shift)); };
    auto row_at = [&](uint32_t at) { return a.idx ? a.idx[at] : at; };
    // new entries: the next round's ids and row numbers, the positions of the one behind it
    unsigned int p = first, left = (count - first + step - 1) / step;          // their first one, how many rounds of them are left
    uint32_t at1 = position(p), at2 = position(left > 1u ? p + step : p), row1 = row_at(at1);
    uint2 ids1 = ids_of(at1);
    int parity = 0;
    // The next round: entries that wait where they fill one, the last ones first, or (end) where none is in hand whose entries could join them;
    // otherwise new ones.  Its rows are on their way afterwards.  Returns how many entries it has.
    auto next_round = [&](bool& waited, bool end) -> unsigned int {
        waited = waiting >= (unsigned)ROUND || left == 0u;
        unsigned int n;
        if (waited) {
            n = waiting < (unsigned)ROUND ? waiting : (unsigned)ROUND;
            if (n == 0u || (n < (unsigned)ROUND && !end)) return 0u;
            waiting -= n;
            if (lane < ROUND) {
                const unsigned int q = waiting + ((unsigned)lane < n ? (unsigned)lane : 0u);
                info[parity * ROUND + lane] = later[q];
                info_row[parity * ROUND + lane] = later_row[q];
            }
        } else {
            n = count - p < (unsigned)ROUND ? count - p : (unsigned)ROUND;
            const uint2 ids2 = ids_of(at2);
            const uint32_t row2 = row_at(at2), at3 = position(left > 2u ? p + 2u * step : p);
            if (lane < ROUND) {
                info[parity * ROUND + lane] = make_uint4(ids1.x, ids1.y, at1, 0u);
                info_row[parity * ROUND + lane] = row1;
            }
            ids1 = ids2;
            row1 = row2;
            at1 = at2;
            at2 = at3;
            p += step;
            --left;
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int u = 0; u < EACH; ++u) {
            const int q = parity * ROUND + GROUPS * u + grp;
            fetch(u, info[q].x, info_row[q]);
        }
        return n;
    };
    bool waited;
    unsigned int n = next_round(waited, false);
    while (n != 0u) {
        // this round's differences to LDS, the next one's rows on their way
#pragma unroll
        for (int u = 0; u < EACH; ++u) lay(u);
        const uint4* const mine = info + parity * ROUND;
        const bool old = waited;
        const unsigned int m = n;
        parity ^= 1;
        n = next_round(waited, false);
        __builtin_amdgcn_wave_barrier();
        const uint4 my = mine[e];
        const unsigned int word = old ? my.w >> 24 : 0u;               // of its ids
        const uint32_t at = old ? my.y : my.z;
        bd = old ? __uint_as_float(my.z) : INFINITY;
        bk = old ? (int)(my.w & kNoRow) : 0x7fffffff;
        sum(my.x);
        const bool here = lane < 2 * (int)m && c == 0;
        unsigned int rest_of = 0xffffffffu;
        if (!old) rest_of = here ? my.y : 0xffffffffu;
        else if (here && word + 1u < 1u << pair_shift && my.x >> 16 != 0xffffu) rest_of = a.pairs[((int64_t)at << pair_shift) + word + 1u];
        const bool more = rest_of != 0xffffffffu;
        if (here && !more && bk < a.K) a.bmu[at] = node_of_row(bk, a.K);
        const unsigned long long wait = __ballot(more);
        if (wait != 0ull) {
            const unsigned int to = waiting + __builtin_amdgcn_mbcnt_hi((unsigned)(wait >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)wait, 0));
            if (more) {
                later[to] = make_uint4(rest_of, at, __float_as_uint(bd), ((unsigned)bk & kNoRow) | (word + 1u) << 24);
                later_row[to] = info_row[(parity ^ 1) * ROUND + e];
            }
            waiting += (unsigned)__popcll(wait);
        }
        __builtin_amdgcn_wave_barrier();
        if (n == 0u) n = next_round(waited, true);          // (the last rounds' entries that wait; each entry comes four times at most)
    }
}

template <bool PAIRS>
__global__ void __launch_bounds__(kExactThreads) __attribute__((amdgpu_waves_per_eu(4))) bmu_exact_kernel(const BmuArgs a)
{
    // PAIRS: two differences of each entry of the pair list in hand; otherwise only the slab of the listed samples' features
    extern __shared__ float4 lds4[];
    float4 (*xs4)[kExactGroup / 4] = reinterpret_cast<float4 (*)[kExactGroup / 4]>(lds4);   // [feature within a 64-wide slab][sample]
    constexpr int kWaves = kExactThreads / 64;
    __shared__ float red_d[kWaves][kExactGroup];
    __shared__ int red_k[kWaves][kExactGroup];
    float* xs = reinterpret_cast<float*>(xs4);
    const float* __restrict__ wt = a.wt;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    // the whole list, or what the candidate pass left over
    const unsigned int listed = a.scal[a.slot];
    const bool by_cand = a.second_only || cand_pass_serves(a, listed);
    const unsigned int count = by_cand ? a.scal[a.slot2] : listed;
    const uint32_t* __restrict__ list = by_cand ? a.recheck2 : a.recheck;
    if (blockIdx.x == 0 && tid == 0) {
        // running total over the calls that share one weight preparation (the split search for D <= 64 counts its near
        // ties itself)
        if (!a.counts_near) atomicAdd(&a.scal[3], listed);
        a.scal[26 - a.slot] = 0u;       // the next call counts into the other slots (12, 13 and 14, 15; 4 and 5)
        a.scal[27 - a.slot] = 0u;
        a.scal[9 - a.slot2] = 0u;
    }
    if (PAIRS && a.tops && blockIdx.x == 0 && tid < kTops) {   // the search has read its maxima: kept for later passes, zero again for the next preparation
        a.tops[kTopsKept + tid] = a.tops[tid];
        a.tops[tid] = 0u;
    }
    double qs = 0.0, qs2 = 0.0;
    if constexpr (PAIRS) {
        switch (pair_lanes(a.D)) {
        case 4: pair_list<4>(a, lds4); break;
        case 8: pair_list<8>(a, lds4); break;
        default: pair_list<16>(a, lds4); break;
        }
    }
    // (PAIRS: from the last workgroup on, so that a short list goes to workgroups without pairs: the kernel 17.5 -> 13.6 us at
    // 250,000 x 37, together with half as many workgroups.  Two fit a compute unit.)
    for (unsigned int g0 = (PAIRS ? gridDim.x - 1 - blockIdx.x : blockIdx.x) * kExactGroup; g0 < count; g0 += gridDim.x * kExactGroup) {
        float bestd[kExactGroup];
        int bestk[kExactGroup];
#pragma unroll
        for (int s = 0; s < kExactGroup; ++s) {
            bestd[s] = INFINITY;
            bestk[s] = 0x7fffffff;
        }
        auto sweep = [&](auto nodes) {
            constexpr int NODES = decltype(nodes)::value;
            for (int kb = 0; kb < a.kpad; kb += kExactThreads * NODES) {
                float dist[kExactGroup][NODES];
#pragma unroll
                for (int s = 0; s < kExactGroup; ++s)
#pragma unroll
                    for (int u = 0; u < NODES; ++u) dist[s][u] = 0.f;
                for (int d0 = 0; d0 < a.D; d0 += 64) {
                    const int dn = (a.D - d0 < 64) ? a.D - d0 : 64;
                    __syncthreads();
                    for (int e = tid; e < kExactGroup * dn; e += kExactThreads) {
                        const int s = e / dn, d = e % dn;
                        const unsigned int ge = (g0 + s < count) ? g0 + s : count - 1;
                        const int64_t i = (int64_t)list[ge];
                        const int64_t r = a.idx ? (int64_t)a.idx[i] : i;
                        xs[d * kExactGroup + s] = a.X[r * a.ldx + d0 + d];
                    }
                    __syncthreads();
                    // Eight features at a time: their sixteen weight loads are in flight together (no condition on any: with one
                    // branch per load the compiler kept them apart, and the pass took twice as long on a 4096-node map).
                    constexpr int kAtOnce = 8;
                    const float* wcol[NODES];
#pragma unroll
                    for (int u = 0; u < NODES; ++u) {
                        const int k = kb + u * kExactThreads + tid;
                        wcol[u] = wt + (size_t)d0 * a.kpad + (k < a.kpad ? k : a.kpad - 1);
                    }
                    auto add = [&](int d, const float (&w)[NODES]) {
                        float xv[kExactGroup];
#pragma unroll
                        for (int q = 0; q < kExactGroup / 4; ++q) {
                            const float4 v4 = xs4[d][q];
                            xv[4 * q + 0] = v4.x;
                            xv[4 * q + 1] = v4.y;
                            xv[4 * q + 2] = v4.z;
                            xv[4 * q + 3] = v4.w;
                        }
#pragma unroll
                        for (int s = 0; s < kExactGroup; ++s)
#pragma unroll
                            for (int u = 0; u < NODES; ++u) {
                                const float df = xv[s] - w[u];
                                dist[s][u] = fmaf(df, df, dist[s][u]);
                            }
                    };
                    int d = 0;
                    for (; d + kAtOnce <= dn; d += kAtOnce) {
                        float w[kAtOnce][NODES];
#pragma unroll
                        for (int t = 0; t < kAtOnce; ++t)
#pragma unroll
                            for (int u = 0; u < NODES; ++u) w[t][u] = wcol[u][(size_t)(d + t) * a.kpad];
#pragma unroll
                        for (int t = 0; t < kAtOnce; ++t) add(d + t, w[t]);
                    }
                    for (; d < dn; ++d) {
                        float w[NODES];
#pragma unroll
                        for (int u = 0; u < NODES; ++u) w[u] = wcol[u][(size_t)d * a.kpad];
                        add(d, w);
                    }
                }
#pragma unroll
                for (int u = 0; u < NODES; ++u) {
                    // (PAIRS: the transposed copy is in the stages' order; a thread's columns are of rising stages, so of rising nodes)
                    const int col = kb + u * kExactThreads + tid, k = PAIRS ? node_of_row(col, a.K) : col;
#pragma unroll
                    for (int s = 0; s < kExactGroup; ++s)
                        if (col < a.K && dist[s][u] < bestd[s]) {
                            bestd[s] = dist[s][u];
                            bestk[s] = k;
                        }
                }
            }
        };
        // (a map of up to as many nodes as threads: one each, 2,500 entries on 400 nodes x 25 take 20 us instead of 22)
        if (a.kpad <= kExactThreads) sweep(std::integral_constant<int, 1>{});
        else sweep(std::integral_constant<int, kExactNodesPerThread>{});
        // lowest distance, then lowest node index, across the workgroup
#pragma unroll
        for (int s = 0; s < kExactGroup; ++s) {
            float bd = bestd[s];
            int bk = bestk[s];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const float od = __shfl_xor(bd, o);
                const int ok = __shfl_xor(bk, o);
                if (od < bd || (od == bd && ok < bk)) {
                    bd = od;
                    bk = ok;
                }
            }
            if (lane == 0) {
                red_d[wave][s] = bd;
                red_k[wave][s] = bk;
            }
        }
        __syncthreads();
        if (tid < kExactGroup && g0 + tid < count) {
            float bd = red_d[0][tid];
            int bk = red_k[0][tid];
            for (int w = 1; w < kWaves; ++w) {
                const float od = red_d[w][tid];
                const int ok = red_k[w][tid];
                if (od < bd || (od == bd && ok < bk)) {
                    bd = od;
                    bk = ok;
                }
            }
            if (bk >= a.K) bk = 0; // only reachable with non-finite input
            const int64_t i = (int64_t)list[g0 + tid];
            a.bmu[i] = bk;
            if (a.d2) a.d2[i] = bd;
            qs += sqrt((double)bd);
            qs2 += (double)bd;
        }
    }
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

// ---------------------------------------------------------------------------------------------------------
// Distances to the winners, where they are asked for, for rows of up to 4 LPR <= 64 features: direct differences on the values
// as given.  Bound by memory: a wavefront takes 64 consecutive samples, LPR lanes a row (16 bytes each, and the winner's row
// from L2), up to eight rows of each group in flight; lane `sub` of a group keeps the sum of its sub-th sample, so units, row
// numbers, distances and the square roots are one coalesced access, or one instruction, per 64 samples.
// 900,000 listed rows of 25 features 30 us, 250,000 x 37 12 us.  (At the end of the search's tiles, where the rows were read again
// before, it took 28 and 6 us of the search, and for samples near their node values that the centrings had rounded.)
// ---------------------------------------------------------------------------------------------------------
constexpr int kDistThreads = 256;

template <int LPR>
__global__ void __launch_bounds__(kDistThreads) bmu_distance_kernel(const BmuArgs a)
{
    constexpr int U = LPR < 8 ? LPR : 8;
    const int lane = threadIdx.x & 63, sub = lane & (LPR - 1), group = lane & ~(LPR - 1);
    const int start = 4 * sub < a.D - 4 ? 4 * sub : a.D - 4, shift = 4 * sub - start;      // own elements of the window: >= shift
    const int64_t units = (a.m + 63) / 64, step = (int64_t)gridDim.x * (kDistThreads / 64);
    double qs = 0.0, qs2 = 0.0;
    auto sample = [&](int64_t unit) {
        const int64_t i = unit * 64 + lane;
        return i < a.m ? i : a.m - 1;
    };
    int64_t unit = (int64_t)blockIdx.x * (kDistThreads / 64) + (threadIdx.x >> 6);
    int node = 0;
    uint32_t row = 0;
    if (unit < units) {
        const int64_t i = sample(unit);
        node = a.bmu[i];
        row = a.idx ? a.idx[i] : (uint32_t)i;
    }
    for (; unit < units; unit += step) {
        const int64_t next = sample(unit + step < units ? unit + step : unit);
        const int node_next = a.bmu[next];
        const uint32_t row_next = a.idx ? a.idx[next] : (uint32_t)next;
        node = (node >= 0 && node < a.K) ? node : 0;
        float mine = 0.0f;
#pragma unroll
        for (int b = 0; b < LPR; b += U) {
            float4 x[U], w[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t r = __shfl(row, group + b + u);
                const int k = __shfl(node, group + b + u);
                x[u] = load4(a.X + (int64_t)r * a.ldx + start);
                w[u] = load4(a.W + (size_t)k * a.D + start);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float d0 = shift <= 0 ? x[u].x - w[u].x : 0.0f, d1 = shift <= 1 ? x[u].y - w[u].y : 0.0f;
                const float d2 = shift <= 2 ? x[u].z - w[u].z : 0.0f, d3 = shift <= 3 ? x[u].w - w[u].w : 0.0f;
                float d = d0 * d0;
                d = fmaf(d1, d1, d);
                d = fmaf(d2, d2, d);
                d = fmaf(d3, d3, d);
#pragma unroll
                for (int o = LPR / 2; o > 0; o >>= 1) d += __shfl_xor(d, o);
                mine = sub == b + u ? d : mine;
            }
        }
        const int64_t i = unit * 64 + lane;
        if (i < a.m) {
            if (a.d2) a.d2[i] = mine;
            if (a.qe) {
                qs += sqrt((double)mine);
                qs2 += (double)mine;
            }
        }
        node = node_next;
        row = row_next;
    }
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

// qe[0..1] += the call's partial sums, scal[3] += its near ties; the slots are left zero for the next call
__global__ void __launch_bounds__(kQeSlots) qe_finish_kernel(double* __restrict__ part, double* __restrict__ qe,
                                                             unsigned int* __restrict__ scal)
{
    __shared__ double w[kQeSlots / 64][3];
    const int tid = threadIdx.x;
    double s0 = part[2 * tid], s1 = part[2 * tid + 1], s2 = part[2 * kQeSlots + tid];
    part[2 * tid] = 0.0;
    part[2 * tid + 1] = 0.0;
    part[2 * kQeSlots + tid] = 0.0;
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if ((tid & 63) == 0) {
        w[tid >> 6][0] = s0;
        w[tid >> 6][1] = s1;
        w[tid >> 6][2] = s2;
    }
    __syncthreads();
    if (tid == 0) {
        double t0 = 0.0, t1 = 0.0, t2 = 0.0;
        for (int q = 0; q < kQeSlots / 64; ++q) {
            t0 += w[q][0];
            t1 += w[q][1];
            t2 += w[q][2];
        }
        qe[0] += t0;
        qe[1] += t1;
        scal[3] += (unsigned int)t2;
    }
}

// ---------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------
static int steps_for(int D)
{
    const int need = (D + 1) / 2;
    const int avail[] = {4, 8, 12, 16, 20, 25, 28, 32};   // MFMA steps per block; the smallest that holds D
    for (int s : avail)
        if (need <= s) return s;
    return 0;
}

int launch_fill_zero(som_ctx* ctx, void* p, size_t bytes)
{
    if (bytes == 0) return SOM_OK;
    const size_t words = bytes / 4;
    int blocks = (int)((words + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, ctx->stream, (uint32_t*)p, words);
    return check_hip(ctx, hipGetLastError(), "fill_zero launch");
}

// Whether a search for up to 64 features takes half-precision and fp6 parts, or two bf16 parts.  The former need `fewer` MFMAs less for a block
// of 32 nodes, but their samples cost more to cut (10 to 13 us for 10^6 rows), their preparation 2 us more, and their wider bound lists about
// twice as many samples, up to 10 us even where those are few.  Whole searches, two bf16 parts and these: on 400 nodes, 10^6 x 25 120 us
// and 121, 10^6 x 50 166 and 161; on 256 nodes 10^6 x 25 89 and 96, 10^6 x 56 144 and 135; on 1024 nodes 120,000 x 50 66 and 68, 250,000 x 56
// 117 and 103, 10^6 x 25 233 and 200, 10^6 x 50 343 and 317, 10^6 x 64 398 and 331; 500,000 x 50 on 2500 395 and 361.  Up to 20 features
// they save one MFMA or none and lose on every map (10^6 x 16 on 1024 nodes 168 and 180, 10^6 x 20 on 400 108 and 122).
// (rows: of the whole epoch, also where they come in chunks.  The forms list different samples, and of nodes that float32 differences cannot tell
// apart a listed one may get another than a score would give it: an epoch's units must not depend on the length of its chunks.)
static bool half_parts_pay(int32_t K, int32_t D, int64_t rows)
{
    if (D <= 20) return false;
    const int left = D % 16, two_parts = left >= 1 && left <= 4 ? 3 * (D / 16) + 1 : 3 * ((D + 15) / 16);
    const int64_t fewer = (int64_t)((K + 31) / 32) * (two_parts - (D + 31) / 32 - (half_norm_group(D) / 4 + 1));
    return fewer >= 40 && rows * fewer >= 40000000;
}

int bmu_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, int64_t rows, int64_t all, BmuPrep* out, double* qe, int32_t* small)
{
    int steps, nch;
    if (D <= 2 * kMaxStepsResident) {
        steps = steps_for(D);
        nch = 1;
    } else {
        // chunk width 50, 56 or 64 features, whichever wastes least (a chunk costs about three MFMA steps of
        // overhead); the wider one on a tie
        steps = 0;
        nch = 0;
        for (int cand : {32, 28, 25}) {
            const int n = (D + 2 * cand - 1) / (2 * cand);
            if (steps == 0 || n * (cand + 3) < nch * (steps + 3)) {
                steps = cand;
                nch = n;
            }
        }
    }
    const int stride = 2 * steps + 1;
    const int kpad = ((K + kNodesPerStage - 1) / kNodesPerStage) * kNodesPerStage;
    const bool wide_split = D > 2 * kMaxStepsResident && K > kSplitMinNodes && ctx->search != SOM_SEARCH_FLOAT32;
    out->form = wide_split ? bmu_wide_form(ctx, K, D, rows) : 0;
    const bool no_stage = wide_split || (D >= 4 && K > kSplitMinNodes && ctx->search != SOM_SEARCH_FLOAT32);
    const size_t stage_bytes = no_stage ? 0 : (size_t)(kpad / kNodesPerStage) * nch * stage_floats_for(stride) * sizeof(float);
    const size_t wt_bytes = (size_t)D * kpad * sizeof(float) + 255 & ~(size_t)255;
    // the centre vector is zero-padded to whole chunks (and to the 64 entries the resident kernel reads)
    const size_t centre_floats = (size_t)(nch > 1 ? nch * 2 * steps : 64);
    const size_t centre_bytes = ((centre_floats > (size_t)D ? centre_floats : (size_t)D) * sizeof(float) + 255) / 256 * 256;
    // rows for the bf16 matrix pipe where the split search applies
    const bool split = D >= 4 && K > kSplitMinNodes && ctx->search != SOM_SEARCH_FLOAT32;
    // D <= 64: half-precision and fp6 parts, the norms in four places behind the features; narrow rows two bf16 parts
    const bool half = split && nch == 1 && half_parts_pay(K, D, all);
    const int units = half ? (D + 31) / 32 : 0, tail_r = split && nch == 1 && !half && D % 16 >= 1 && D % 16 <= 4 ? D % 16 : 0;
    const int kb = !split || nch > 1 ? 0 : half ? half_norm_group(D) / 4 + 1 : tail_r ? D / 16 : (D + 15) / 16;
    const int form = units ? kFormHalf1 + units - 1 : tail_r ? kFormTail : kb == 4 && K <= kFewNodes ? kFormFew : kFormWhole;
    if (!wide_split) out->form = form;
    // (D > 64: rows in the order of the form that the call takes)
    const size_t stage16_one = (split && nch == 1) ? (size_t)split_stage_f4(kb, form) * 16 : 0;
    const size_t stage16_bytes = !split ? 0 : nch == 1 ? (size_t)(kpad / kNodesPerStage) * stage16_one : bmu_wide_blob_bytes(out->form, K, D, kpad);
    const size_t wrow_bytes = (split && nch == 1) ? (size_t)K * D * sizeof(float) : 0;
    const size_t need = stage_bytes + wt_bytes + centre_bytes + stage16_bytes + wrow_bytes + 256;
    if (need > ctx->prep_bytes) {
        if (ctx->prep_blob) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->prep_blob);
            ctx->prep_blob = nullptr;
            ctx->prep_bytes = 0;
        }
        if (hipMalloc(&ctx->prep_blob, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the weight workspace", need);
        }
        ctx->prep_bytes = need;
        ctx->prep_clean = false;
    }
    char* base = (char*)ctx->prep_blob;
    out->scal = (unsigned int*)base;
    out->tops = (unsigned int*)(base + 128);
    out->stage = (float*)(base + 256);
    out->wt = (float*)(base + 256 + stage_bytes);
    out->centre = (float*)(base + 256 + stage_bytes + wt_bytes);
    out->stage16 = split ? (void*)(base + 256 + stage_bytes + wt_bytes + centre_bytes) : nullptr;
    out->tail_r = tail_r;
    out->wrow = wrow_bytes ? (float*)(base + 256 + stage_bytes + wt_bytes + centre_bytes + stage16_bytes) : nullptr;
    out->kb = kb;
    out->kpad = kpad;
    out->steps = steps;
    out->stride = stride;
    out->nch = nch;
    out->calls = 0;
    if (split && nch == 1) {
        // (after a new allocation, or a call that failed between here and its last kernel)
        if (!ctx->prep_clean)
            if (int rc = launch_fill_zero(ctx, out->tops, 64)) return rc;
        ctx->prep_clean = false;
        HalfPrep sp{};
        sp.stage16 = (char*)out->stage16;
        sp.wrow = out->wrow;
        sp.kb_count = kb;
        sp.tail_r = tail_r;
        sp.units = units;
        sp.row_bytes = split_row_bytes(kb, form);
        sp.stage16_bytes = (int)stage16_one;
        const dim3 grid((unsigned)(kpad / kPrepNodes)), block(64 * kPrepNodes);
        if (half) {
            void (*kernel)(const float*, int, int, int, float*, float*, unsigned int*, unsigned int*, double*, int32_t*, const HalfPrep) = bmu_split_prep_kernel;
            hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, W, K, D, kpad, out->centre, out->wt, out->scal, out->tops, qe, small, sp);
        } else {
            void (*kernel)(const float*, int, int, int, float*, float*, unsigned int*, unsigned int*, double*, int32_t*, const SplitPrep) = bmu_split_prep_kernel;
            hipLaunchKernelGGL(kernel, grid, block, 0, ctx->stream, W, K, D, kpad, out->centre, out->wt, out->scal, out->tops, qe, small, (const SplitPrep&)sp);
        }
        return check_hip(ctx, hipGetLastError(), "bmu (split) preparation launch");
    }
    hipLaunchKernelGGL(bmu_centre_kernel, dim3((unsigned)(centre_bytes / 256)), dim3(1024), 0, ctx->stream, W, K, D,
                       out->centre, out->scal, wide_split ? bmu_wide_spread(*out, K, D) : nullptr, small);
    if (wide_split) {
        if (int rc = check_hip(ctx, hipGetLastError(), "bmu_centre launch")) return rc;
        return bmu_wide_prepare(ctx, W, K, D, *out, qe, small);
    }
    // one thread per element of the padded stage matrix and of the transposed copy, one wavefront per four nodes
    long long elems = (long long)kpad * nch * stride;
    if (elems < (long long)kpad * 16) elems = (long long)kpad * 16;
    if (elems < (long long)kpad * D) elems = (long long)kpad * D;
    hipLaunchKernelGGL(bmu_prep_kernel, dim3((unsigned)((elems + 255) / 256)), dim3(256), 0, ctx->stream, W, K, D, kpad, stride, nch,
                       stage_floats_for(stride), out->centre, out->stage, out->wt, out->scal, qe, small);
    return check_hip(ctx, hipGetLastError(), "bmu_prep launch");
}

template <int STEPS>
static int launch_bmu_wide(som_ctx* ctx, const BmuArgs& a)
{
    constexpr size_t lds_bytes = 2 * (size_t)stage_floats_for(2 * STEPS + 1) * sizeof(float);
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    auto kern = bmu_wide_kernel<STEPS>;
    if (!attr_set) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    const int64_t per_group = (int64_t)kWavesPerGroup * 32;
    const int64_t groups = (a.m + per_group - 1) / per_group;
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kThreads), lds_bytes, ctx->stream, a);
    return check_hip(ctx, hipGetLastError(), "bmu (wide) kernel launch");
}

// grid of the candidate kernels: the tiles of the longest list they may serve, at most kCandGrid workgroups
static unsigned cand_grid(const BmuArgs& a, int64_t per_tile)
{
    const int64_t most = a.m < (int64_t)a.cand_cap ? a.m : (int64_t)a.cand_cap;
    const int64_t tiles = (most + per_tile - 1) / per_tile;
    return (unsigned)(tiles < kCandGrid ? tiles : kCandGrid);
}

template <int STEPS>
static int launch_bmu_wide_cand(som_ctx* ctx, const BmuArgs& a)
{
    constexpr size_t lds_bytes = 2 * (size_t)stage_floats_for(2 * STEPS + 1) * sizeof(float);
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    auto kern = bmu_wide_cand_kernel<STEPS>;
    if (!attr_set) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(cand_grid(a, (int64_t)kWavesPerGroup * 32)), dim3(kThreads), lds_bytes, ctx->stream, a);
    return check_hip(ctx, hipGetLastError(), "bmu (wide) candidate kernel launch");
}

template <int STEPS, int MS>
static int launch_bmu_cand(som_ctx* ctx, const BmuArgs& a)
{
    constexpr size_t lds_bytes = 2 * (size_t)stage_floats_for(2 * STEPS + 1) * sizeof(float);
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    auto kern = bmu_cand_kernel<STEPS, MS>;
    if (!attr_set) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(cand_grid(a, (int64_t)kWavesPerGroup * MS * 32)), dim3(kThreads), lds_bytes, ctx->stream,
                       a);
    return check_hip(ctx, hipGetLastError(), "bmu candidate kernel launch");
}

static int dispatch_bmu_cand(som_ctx* ctx, int steps, const BmuArgs& a)
{
    switch (steps) {
    case 4: return launch_bmu_cand<4, 2>(ctx, a);
    case 8: return launch_bmu_cand<8, 2>(ctx, a);
    case 12: return launch_bmu_cand<12, 2>(ctx, a);
    case 16: return launch_bmu_cand<16, 2>(ctx, a);
    case 20: return launch_bmu_cand<20, 2>(ctx, a);
    case 25: return launch_bmu_cand<25, 2>(ctx, a);
    case 28: return launch_bmu_cand<28, 2>(ctx, a);
    case 32: return launch_bmu_cand<32, 2>(ctx, a);
    }
    return fail(ctx, SOM_EINVAL, "no BMU kernel for %d steps", steps);
}

template <int STEPS, int MS>
static int launch_bmu(som_ctx* ctx, const BmuArgs& a)
{
    constexpr int STRIDE = 2 * STEPS + 1;
    constexpr size_t lds_bytes = 2 * (size_t)stage_floats_for(STRIDE) * sizeof(float);
    // maps that end in whole blocks of padding nodes take the variant that skips them
    const bool pad = a.kpad - a.K >= 32;
    static bool attr_set_dev[kMaxDevices][2] = {};    // the attribute belongs to the device, not to the process
    bool* attr_set = attr_set_dev[ctx->device];
    auto kern = pad ? bmu_kernel<STEPS, MS, true> : bmu_kernel<STEPS, MS, false>;
    if (!attr_set[pad]) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set[pad] = true;
    }
    // Two workgroups fit a compute unit, so the grid runs in rounds of 2 * units tiles and a unit's time in the
    // last, partial round goes with the number of sample blocks it gets.  When halving the tiles of that round
    // lowers the largest share (measured at 10^6 samples on 256 units: 7.63 rounds cost as much as 8), they are
    // halved.
    const int64_t per_group = (int64_t)kWavesPerGroup * MS * 32;
    const int64_t tiles = (a.m + per_group - 1) / per_group;
    const int64_t units = ctx->units, rem = tiles % (2 * units);
    BmuArgs b = a;
    b.full_tiles = tiles;
    int64_t groups = tiles;
    if (MS > 1 && tiles >= 2 * units && rem > 0 && (2 * rem + units - 1) / units < 2 * ((rem + units - 1) / units)) {
        b.full_tiles = tiles - rem;
        const int64_t left = a.m - b.full_tiles * per_group, per_half = per_group / 2;
        groups = b.full_tiles + (left + per_half - 1) / per_half;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kThreads), lds_bytes, ctx->stream, b);
    return check_hip(ctx, hipGetLastError(), "bmu kernel launch");
}

template <int KB, int FORM, int MS>
static int launch_bmu_split(som_ctx* ctx, const BmuArgs& a)
{
    constexpr size_t lds_bytes = 2 * (size_t)split_pitch(KB, FORM) + 6 * kThreads * sizeof(float);
    static_assert(lds_bytes + 512 <= 80 * 1024, "two workgroups per compute unit");
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    auto kern = bmu_split_kernel<KB, FORM, MS>;
    if (!attr_set) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    // full tiles, and half tiles for the last partial round where that lowers the largest share (as launch_bmu)
    const int64_t per_group = (int64_t)kWavesPerGroup * MS * 32;
    const int64_t tiles = (a.m + per_group - 1) / per_group;
    const int64_t units = ctx->units, rem = tiles % (2 * units);
    BmuArgs b = a;
    b.full_tiles = tiles;
    int64_t groups = tiles;
    if (MS > 1 && tiles >= 2 * units && rem > 0 && (2 * rem + units - 1) / units < 2 * ((rem + units - 1) / units)) {
        b.full_tiles = tiles - rem;
        const int64_t left = a.m - b.full_tiles * per_group, per_half = per_group / 2;
        groups = b.full_tiles + (left + per_half - 1) / per_half;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)groups), dim3(kThreads), lds_bytes, ctx->stream, b);
    return check_hip(ctx, hipGetLastError(), "bmu split kernel launch");
}

template <int KB, int FORM, int MS>
static int launch_bmu_split_cand(som_ctx* ctx, const BmuArgs& a)
{
    constexpr size_t lds_bytes = cand_lds(KB, FORM);
    static_assert(lds_bytes <= 80 * 1024, "two workgroups per compute unit");
    static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
    bool& attr_set = attr_set_dev[ctx->device];
    auto kern = bmu_split_cand_kernel<KB, FORM, MS>;
    if (!attr_set) {
        if (int rc = check_hip(ctx,
                               hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes),
                               "raising the dynamic LDS limit"))
            return rc;
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(cand_grid(a, (int64_t)kWavesPerGroup * MS * 32)), dim3(kThreads), lds_bytes, ctx->stream,
                       a);
    return check_hip(ctx, hipGetLastError(), "bmu split candidate kernel launch");
}

// calls launch with the (blocks, form) of a row as types
template <typename F>
static int dispatch_split(som_ctx* ctx, int kb, int form, F&& launch)
{
#define SOM_SPLIT_CASE(KB, FORM) \
    if (kb == KB && form == FORM) return launch(std::integral_constant<int, KB>{}, std::integral_constant<int, FORM>{});
    SOM_SPLIT_CASE(0, kFormTail)
    SOM_SPLIT_CASE(1, kFormWhole)
    SOM_SPLIT_CASE(1, kFormTail)
    SOM_SPLIT_CASE(2, kFormWhole)
    SOM_SPLIT_CASE(2, kFormTail)
    SOM_SPLIT_CASE(3, kFormWhole)
    SOM_SPLIT_CASE(3, kFormTail)
    SOM_SPLIT_CASE(4, kFormWhole)
    SOM_SPLIT_CASE(4, kFormFew)
    SOM_SPLIT_CASE(2, kFormHalf1)
    SOM_SPLIT_CASE(3, kFormHalf1)
    SOM_SPLIT_CASE(3, kFormHalf2)
    SOM_SPLIT_CASE(4, kFormHalf2)
    SOM_SPLIT_CASE(5, kFormHalf2)
#undef SOM_SPLIT_CASE
    return fail(ctx, SOM_EINVAL, "no split BMU kernel for %d blocks of form %d", kb, form);
}

static int dispatch_bmu_split(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a)
{
    return dispatch_split(ctx, prep.kb, prep.form, [&](auto kb, auto form) { return launch_bmu_split<kb, form, kSplitMS>(ctx, a); });
}

static int dispatch_bmu_split_cand(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a)
{
    return dispatch_split(ctx, prep.kb, prep.form, [&](auto kb, auto form) { return launch_bmu_split_cand<kb, form, kSplitMS>(ctx, a); });
}

static int dispatch_bmu(som_ctx* ctx, int steps, const BmuArgs& a)
{
    switch (steps) {
    case 4: return launch_bmu<4, 2>(ctx, a);
    case 8: return launch_bmu<8, 2>(ctx, a);
    case 12: return launch_bmu<12, 2>(ctx, a);
    case 16: return launch_bmu<16, 2>(ctx, a);
    case 20: return launch_bmu<20, 2>(ctx, a);
    case 25: return launch_bmu<25, 2>(ctx, a);
    case 28: return launch_bmu<28, 2>(ctx, a);
    case 32: return launch_bmu<32, 2>(ctx, a);
    }
    return fail(ctx, SOM_EINVAL, "no BMU kernel for %d steps", steps);
}

static int launch_bmu_distances(som_ctx* ctx, const BmuArgs& a)
{
    const int64_t groups = (a.m + kDistThreads - 1) / kDistThreads;
    const dim3 grid((unsigned)(groups < 2048 ? groups : 2048)), block(kDistThreads);
    if (a.D <= 16)
        hipLaunchKernelGGL(bmu_distance_kernel<4>, grid, block, 0, ctx->stream, a);
    else if (a.D <= 32)
        hipLaunchKernelGGL(bmu_distance_kernel<8>, grid, block, 0, ctx->stream, a);
    else
        hipLaunchKernelGGL(bmu_distance_kernel<16>, grid, block, 0, ctx->stream, a);
    return check_hip(ctx, hipGetLastError(), "bmu distance launch");
}

static int bmu_run_pass(som_ctx* ctx, BmuPrep& prep, BmuArgs a);

// what a pass's workspaces can have
static size_t memory_left(som_ctx* ctx)
{
    size_t left = 0, total = 0;
    if (hipMemGetInfo(&left, &total) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    const size_t sets = ctx->recheck_sets ? (ctx->recheck_cap < kCandCapMax ? ctx->recheck_cap : kCandCapMax) * 2 * sizeof(ulonglong2) : 0;
    return left + ctx->recheck_cap * 12 + sets + ctx->pairs_bytes + ctx->parts_bytes;
}

// The rows go through in passes of at most 2^27 (rows of more than 64 features: bmu_wide_pass_rows), and of fewer where memory runs out.  The
// re-decision workspace then stays at 3.8 GB whatever m is (28 bytes a row on maps of kPairMany nodes and more, 20 on others, 12 and the candidate
// sets, 0.5 GB, in the float32 searches), and a pass's list stays within what the candidate pass can hold (2^24 entries, an eighth of a
// pass) — one call over 10^9 rows listed more than that and fell back to direct differences over all nodes for every listed sample.
// A search that memory kept from its passes starts with the rows that it held when it comes again, unless more memory is left than then: a
// failing allocation costs a wait for the stream and the workspace that served the last call.
int bmu_run(som_ctx* ctx, BmuPrep& prep, BmuArgs a)
{
    int64_t kRowsPerPass = (int64_t)1 << 27;
    const int64_t m = a.m;
    const bool wide_split = prep.stage16 && prep.nch > 1;
    if (wide_split) kRowsPerPass = bmu_wide_pass_rows(prep, a.D);
    const int64_t asked = m < kRowsPerPass ? m : kRowsPerPass;
    auto& scarce = ctx->scarce;
    bool fewer = false;
    if (asked == scarce.asked && a.K == scarce.K && a.D == scarce.D) {
        if (memory_left(ctx) <= scarce.left) kRowsPerPass = scarce.held;
        else scarce.asked = 0;
    }
    for (int64_t off = 0; off < m;) {
        BmuArgs b = a;
        b.m = m - off < kRowsPerPass ? m - off : kRowsPerPass;
        if (a.idx)
            b.idx = a.idx + off;
        else
            b.X = a.X + off * a.ldx;
        b.bmu = a.bmu + off;
        if (a.d2) b.d2 = a.d2 + off;
        const int calls = prep.calls;
        const size_t events = ctx->prof_used;
        const int rc = bmu_run_pass(ctx, prep, b);
        if (rc == SOM_ENOMEM && b.m > 256) {         // (nothing of the pass has been launched)
            prep.calls = calls;
            ctx->prof_used = events;
            kRowsPerPass = (b.m / 2 + 127) / 128 * 128;
            fewer = true;
            continue;
        }
        if (rc) return rc;
        off += b.m;
    }
    if (fewer) {                                   // (a call that failed altogether, under capture for instance, says nothing about memory)
        scarce.left = memory_left(ctx);
        scarce.asked = asked;
        scarce.held = kRowsPerPass;
        scarce.K = a.K;
        scarce.D = a.D;
    }
    return SOM_OK;
}

static int bmu_run_pass(som_ctx* ctx, BmuPrep& prep, BmuArgs a)
{
    if (a.m <= 0) return SOM_OK;
    auto cand_cap_for = [](size_t cap) { return cap < kCandCapMax ? cap : kCandCapMax; };
    // (the candidate sets are the float32 searches' only: the split searches decide at the end of their candidate tiles, or
    // keep records of their own)
    const bool sets = prep.stage16 == nullptr;
    if ((size_t)a.m > ctx->recheck_cap || (sets && !ctx->recheck_sets)) {
        if (ctx->recheck) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->recheck);
            ctx->recheck = nullptr;
            ctx->recheck_cap = 0;
            ctx->recheck_sets = false;
        }
        // sample positions [cap], cuts [cap], per-sample cuts [cap], candidate sets [cand_cap][2]; the capacity is a multiple of four
        // entries so that the 16-byte candidate sets stay aligned
        const size_t cap = ((size_t)a.m + 3) / 4 * 4, ccap = cand_cap_for(cap);
        const size_t bytes = cap * 12 + (sets ? ccap * 2 * sizeof(ulonglong2) : 0);
        if (hipMalloc((void**)&ctx->recheck, bytes) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate the %lld-entry recheck list", (long long)a.m);
        }
        ctx->recheck_cap = cap;
        ctx->recheck_sets = sets;
    }
    const size_t pair_words = prep.stage16 && prep.nch == 1 ? (a.K >= kPairMany ? 4 : 2) : 0;
    if (const size_t need = (size_t)a.m * pair_words * sizeof(uint32_t); need > ctx->pairs_bytes) {
        if (ctx->pairs) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->pairs);
            ctx->pairs = nullptr;
            ctx->pairs_bytes = 0;
        }
        if (hipMalloc((void**)&ctx->pairs, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate the %lld-entry pair list", (long long)a.m);
        }
        ctx->pairs_bytes = need;
    }
    a.kpad = prep.kpad;
    a.stage = prep.stage;
    a.stride = prep.stride;
    a.stage16 = prep.stage16;
    a.tail_r = prep.tail_r;
    a.wt = prep.wt;
    a.wrow = prep.wrow;
    a.centre = prep.centre;
    a.scal = prep.scal;
    a.norms = prep.calls == 0 ? prep.tops : prep.tops + kTopsKept;
    a.tops = prep.stage16 && prep.nch == 1 && prep.calls == 0 ? prep.tops : nullptr;
    a.recheck = ctx->recheck;
    a.cutv = (float*)(ctx->recheck + ctx->recheck_cap);
    a.cut_all = (float*)(ctx->recheck + 2 * ctx->recheck_cap);
    a.recheck_end = ctx->recheck + ctx->recheck_cap;
    a.pairs = ctx->pairs;
    // (the per-sample cuts are dead once the lists are made: the second list takes their place)
    a.recheck2 = ctx->recheck + 2 * ctx->recheck_cap;
    a.cand = (ulonglong2*)(ctx->recheck + 3 * ctx->recheck_cap);
    a.cand_cap = (uint32_t)cand_cap_for(ctx->recheck_cap);
    // The candidate pass repeats the search for the listed samples at matrix speed (under a nanosecond per sample
    // at K D = 51200, against 3.8 ns for direct differences over all nodes) but has the latency of a whole tile, so
    // it only serves lists above a minimum length; node ids are 16-bit there.
    const bool cand_possible = a.K > 1 && a.K <= 65536 && a.m > (int64_t)kCandMin;
    a.cand_min = !cand_possible ? 0xffffffffu : prep.stage16 ? kCandMin : kCandMinFloat;
    a.qe_part = ctx->qe_part;
    a.counts_near = prep.stage16 ? 1 : 0;
    // the list length restarts for every call (chunk): calls alternate between two counters, and each call's
    // exact pass clears the counter of the next one
    a.slot = 12 + 2 * (prep.calls & 1);
    a.slot2 = 4 + (prep.calls & 1);
    ++prep.calls;
    hipEvent_t stop = nullptr;
    if (ctx->profiling) {
        if (ctx->prof_used == ctx->prof_events.size()) {
            hipEvent_t e0, e1;
            if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
                return fail(ctx, SOM_EHIP, "event creation failed");
            ctx->prof_events.emplace_back(e0, e1);
        }
        (void)hipEventRecord(ctx->prof_events[ctx->prof_used].first, ctx->stream);
        stop = ctx->prof_events[ctx->prof_used].second;
        ++ctx->prof_used;
    }
    const bool wide_split = prep.stage16 && prep.nch > 1;
    if (wide_split) {
        const size_t need = bmu_wide_work_bytes(ctx, prep, a.K, a.D, a.m);
        if (need > ctx->parts_bytes) {
            if (ctx->parts_blob) {
                if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
                (void)hipFree(ctx->parts_blob);
                ctx->parts_blob = nullptr;
                ctx->parts_bytes = 0;
            }
            if (hipMalloc(&ctx->parts_blob, need) != hipSuccess) {
                (void)hipGetLastError();
                return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the wide search's workspace", need);
            }
            ctx->parts_bytes = need;
        }
        if (int rc = bmu_wide_run(ctx, prep, a, ctx->parts_blob)) return rc;
        if (stop) (void)hipEventRecord(stop, ctx->stream);
        if (a.K > 1) {
            if (int rc = bmu_wide_recheck(ctx, prep, a, ctx->parts_blob)) return rc;
            BmuArgs b = a;                       // what the records left over; the distances come afterwards, for all samples
            b.d2 = nullptr;
            b.qe = nullptr;
            b.second_only = 1;
            hipLaunchKernelGGL(bmu_exact_kernel<false>, dim3(1024), dim3(kExactThreads), kExactLds, ctx->stream, b);
            if (int rc = check_hip(ctx, hipGetLastError(), "bmu exact-pass launch")) return rc;
        }
        if (a.d2 || a.qe)
            if (int rc = bmu_wide_distances(ctx, a)) return rc;
        if (a.qe && !a.qe_later) {
            hipLaunchKernelGGL(qe_finish_kernel, dim3(1), dim3(kQeSlots), 0, ctx->stream, a.qe_part, a.qe, a.scal);
            return check_hip(ctx, hipGetLastError(), "quantisation-error reduction launch");
        }
        return SOM_OK;
    }
    int rc = prep.nch > 1 ? (prep.steps == 25   ? launch_bmu_wide<25>(ctx, a)
                             : prep.steps == 28 ? launch_bmu_wide<28>(ctx, a)
                                                : launch_bmu_wide<32>(ctx, a))
                          : (prep.stage16 ? dispatch_bmu_split(ctx, prep, a) : dispatch_bmu(ctx, prep.steps, a));
    if (rc) return rc;
    if (a.K > 1) {
        const int64_t chunks = (a.m + kListThreads * kListPerThread - 1) / (kListThreads * kListPerThread);
        hipLaunchKernelGGL(bmu_list_kernel, dim3((unsigned)(chunks < 1024 ? chunks : 1024)), dim3(kListThreads), 0, ctx->stream, a);
        if ((rc = check_hip(ctx, hipGetLastError(), "bmu list launch"))) return rc;
    }
    if (stop) (void)hipEventRecord(stop, ctx->stream);
    if (cand_possible) {
        rc = prep.nch > 1 ? (prep.steps == 25   ? launch_bmu_wide_cand<25>(ctx, a)
                             : prep.steps == 28 ? launch_bmu_wide_cand<28>(ctx, a)
                                                : launch_bmu_wide_cand<32>(ctx, a))
                          : (prep.stage16 ? dispatch_bmu_split_cand(ctx, prep, a) : dispatch_bmu_cand(ctx, prep.steps, a));
        if (rc) return rc;
        // (the split search for D <= 64 takes the direct differences over its candidates at the end of the candidate
        // tile itself; the others hand their candidate sets to a kernel of their own)
        if (!(prep.stage16 && prep.nch == 1)) {
            hipLaunchKernelGGL(bmu_cand_exact_kernel, dim3(2048), dim3(256), 0, ctx->stream, a);
            if ((rc = check_hip(ctx, hipGetLastError(), "bmu candidate-distance launch"))) return rc;
        }
    }
    if (a.K > 1) {
        if (prep.stage16 && prep.nch == 1) {
            // (two workgroups of 128 registers a thread fit a compute unit; above 53 features a workgroup's rows take more than 64 KB)
            constexpr size_t kOwn = 2 * 4 * (kExactThreads / 64) * kExactGroup + 16 * 2 * 8 + 16 * 4;      // red_d, red_k and group_qe_add's
            auto rows_of = [](int D) constexpr { return (size_t)(kExactThreads / 64) * pair_lds_f4(D) * 16; };
            static_assert(2 * (rows_of(64) + kOwn) <= 160 * 1024, "LDS of two workgroups");
            const size_t rows = rows_of(a.D), lds = rows > kExactLds ? rows : kExactLds;
            static bool attr_set_dev[kMaxDevices] = {};       // the attribute belongs to the device, not to the process
            bool& attr_set = attr_set_dev[ctx->device];
            if (!attr_set) {
                if ((rc = check_hip(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(bmu_exact_kernel<true>),
                                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)rows_of(64)),
                                    "raising the dynamic LDS limit")))
                    return rc;
                attr_set = true;
            }
            BmuArgs b = a;                       // the distances come afterwards, for all samples
            b.d2 = nullptr;
            b.qe = nullptr;
            hipLaunchKernelGGL(bmu_exact_kernel<true>, dim3(512), dim3(kExactThreads), lds, ctx->stream, b);
        }
        else
            hipLaunchKernelGGL(bmu_exact_kernel<false>, dim3(1024), dim3(kExactThreads), kExactLds, ctx->stream, a);
        if ((rc = check_hip(ctx, hipGetLastError(), "bmu exact-pass launch"))) return rc;
        if (a.tops) ctx->prep_clean = true;
    }
    if (prep.stage16 && (a.d2 || a.qe))
        if ((rc = launch_bmu_distances(ctx, a))) return rc;
    if (a.qe && !a.qe_later) {
        hipLaunchKernelGGL(qe_finish_kernel, dim3(1), dim3(kQeSlots), 0, ctx->stream, a.qe_part, a.qe, a.scal);
        rc = check_hip(ctx, hipGetLastError(), "quantisation-error reduction launch");
    }
    return rc;
}

} // namespace som
