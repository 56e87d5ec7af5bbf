// Best-matching-unit search for rows of more than 256 features (bmu_wide_form): the arithmetic of som_bmu_held.hip, half-precision first
// parts and fp6 cross products, three MFMAs for 32 features where two bf16 parts take six, for rows that no wavefront can hold.
//
// Passes.  bmu_cut_samples_kernel cuts every sample once and leaves its parts in memory, 3.5 bytes a value, in the order of the MFMA's lanes:
// cutting them in the tile again for each 256 nodes takes as long as the products (a row's fp6 conversions and error norms are some 400
// vector instructions a chunk and wavefront).  It is bound by memory: 331 us at 10^5 x 2000 for 1.5 GB.  bmu_cut_split_kernel forms the
// scores of 256 samples x 256 nodes a tile; join and direct differences are those of som_bmu_wide.hip.  For the candidate pass the listed
// rows are cut once more, into blocks of their own (bmu_cut_listed_kernel).
//
// Scales.  As held rows, but for each chunk of 64 features of a row its own; a chunk's products are summed from zero and added to the tile's
// accumulators with the factor that takes them back, so the roundings of a chunk are relative to its own size.
//
// Tile.  Eight wavefronts of 32 samples x 256 nodes each: the samples' parts go straight to registers (28 of them a chunk, the next chunk's
// requested a chunk ahead), the weights' in stages of 64 nodes x 64 features through four buffers in LDS, requested three stages
// ahead (global_load_lds) with one barrier a stage.  What bounds it is the caches: 28 KB a stage and unit, 8 TB/s from L2 at 10^5 x 2000
// on 1024 nodes, where the products by themselves would take 400 us of 730 at the power limit.
//
// Measured, whole search, 10^5 rows on 1024 nodes, against the tile of som_bmu_wide.hip: 300 features 317 -> 229 us, 1000 893 -> 641,
// 2000 1707 -> 1172; on 1296 nodes 403 -> 290, 1233 -> 770, 2450 -> 1421 (of which the short lists, which no longer go through all nodes,
// 35, 130 and 280).
#include "som_bmu_wide.hpp"

#include <math.h>

#include <type_traits>

namespace som {

constexpr int kTileThreads = 512;
constexpr int kCutWaves = kTileThreads / 64;
constexpr int kCutRows = kCutWaves * 32;            // samples of a tile
constexpr int kCutTile = 256;                       // nodes of a tile: four stages of 64 rows, two blocks of 32 each
constexpr int kCutChunk = 64;                       // features of a chunk: two units
constexpr int kCutBlock = 7168;                     // bytes of a block's chunk
constexpr int kCutStage = 2 * kCutBlock;            // and of a stage's
constexpr int kCutStages = 4;                       // buffers in LDS
constexpr int kCutLoads = 2;                        // 1 KB loads of a wavefront and stage
constexpr int kCutAhead = 2;                        // groups of MFMAs between a fragment's read from LDS and its use
constexpr int kCutState = 12;                       // words of running state per lane: best, second, where from of four classes
constexpr size_t kCutLds = kCutStages * (size_t)kCutStage + (size_t)kTileThreads * kCutState * sizeof(float);
static_assert(kCutStages * kCutStage <= 65536, "offsets of global_load_lds below 64 KB");

static int64_t cut_rows(int32_t K) { return ((int64_t)K + kCutTile - 1) / kCutTile * kCutTile; }
// stages that hold a node; a last tile of three takes its fourth, of padding, with it (a chunk's parts then have time to come in: on 144 nodes
// 10^5 x 2000 took 375 us in three stages a tile, on 256 in four 252)
__host__ __device__ inline int cut_stages(int K)
{
    const int n = (K + 63) / 64;
    return n + (n % 4 == 3);
}
static size_t cut_blob(int32_t K, int32_t D) { return (size_t)(cut_rows(K) / 64) * (((size_t)D + kCutChunk - 1) / kCutChunk) * kCutStage; }

// ---------------------------------------------------------------------------------------------------------
// Weight preparation: a wavefront a row of the blocks (node_of_row) cuts it, 512 features at a time, and sums what the cuts leave
// over; the rest of the grid writes the transposed copy that the all-nodes pass reads.
// ---------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) bmu_cut_prep_kernel(const float* __restrict__ W, int K, int D, int kpad, int rows, int nch,
                                                            const float* __restrict__ centre, const float* __restrict__ spread,
                                                            char* __restrict__ blob, float* __restrict__ hats, float* __restrict__ norms,
                                                            float* __restrict__ wt, unsigned int* __restrict__ scal,
                                                            double* __restrict__ qe, int32_t* __restrict__ small)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < 2 && qe) qe[e] = 0.0;
    if (e < 4 && small) small[e] = 0;
    const int node_groups = rows / 4;                          // workgroups that take four rows each
    if ((int)blockIdx.x >= node_groups) {
        const int64_t t = (int64_t)(blockIdx.x - node_groups) * 256 + threadIdx.x;
        if (t < (int64_t)D * kpad) {
            const int f = (int)(t / kpad), k = (int)(t - (int64_t)f * kpad);
            wt[t] = k < K ? W[(size_t)k * D + f] : 0.0f;
        }
        return;
    }
    constexpr int kAtOnce = 512;
    __shared__ __align__(16) _Float16 part[4][2][kAtOnce];
    __shared__ float most[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 4 + wave, k = node_of_row(r, K), R = r & 31;
    float top = 0.0f;
    for (int b = lane; b < (D + 63) / 64; b += 64) top = fmaxf(top, spread[b]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    const int sw = scale_for(top);
    if (e == 0) scal[kScalShift] = (unsigned)sw;
    const float s = power_of_two(sw);
    double nrm = 0.0;
    float lo2 = 0.0f, over = 0.0f, q2 = 0.0f;
    // [node tile][chunk][block of the tile]
    char* const to = blob + (size_t)(r >> 8) * nch * 8 * kCutBlock + (size_t)((r >> 5) & 7) * kCutBlock;
    for (int f_lo = 0; f_lo < nch * kCutChunk; f_lo += kAtOnce) {
#pragma unroll
        for (int i = 0; i < kAtOnce / 64; ++i) {
            // place `slot` of a row: features in fours, the last ones shifted back into the row (own features only, zeros in front of them)
            const int slot = lane + 64 * i, q = (f_lo + slot) >> 2, start = 4 * q < D - 4 ? 4 * q : D - 4, f = start + (slot & 3);
            const float v = (k < K && f >= 4 * q) ? W[(size_t)k * D + f] - centre[f] : 0.0f;
            nrm += (double)v * (double)v;
            const float h = v * s;
            const _Float16 hi = (_Float16)h;
            const float left = h - (float)hi;
            const _Float16 lo = (_Float16)left;
            lo2 = fmaf(left, left, lo2);
            over = fmaf(left - (float)lo, left - (float)lo, over);
            part[wave][0][slot] = hi;
            part[wave][1][slot] = lo;
        }
        __syncthreads();
        {
            const int u = lane >> 2, kb = (lane >> 1) & 1, g = lane & 1, ch = f_lo / kCutChunk + (u >> 1);
            if (ch < nch)
                *reinterpret_cast<uint4*>(to + (size_t)ch * 8 * kCutBlock + (u & 1) * 3072 + kb * 1024 + (g * 32 + R) * 16) =
                    *reinterpret_cast<const uint4*>(&part[wave][0][32 * u + 16 * kb + 8 * g]);
        }
        {
            const int u = lane >> 1, g = lane & 1, ch = f_lo / kCutChunk + (u >> 1);       // (thirty-two lanes)
            if (lane < kAtOnce / 16 && ch < nch) {
                // (the order in which the tile's lanes come by a unit's values: its eights 0, 2, 1 and 3)
                const uint4* from = reinterpret_cast<const uint4*>(&part[wave][g][32 * u]);
                struct {
                    uint4 e[4];
                } eights = {{from[0], from[2], from[1], from[3]}};
                const halfx32 v = __builtin_bit_cast(halfx32, eights);
                const float scale = g == 0 ? power_of_two(kTopBit - 2) : power_of_two(-3);
                const uintx6 q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(v, scale);
                const halfx32 d = __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(q, scale);
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    const float x = (float)v[i] - (float)d[i];
                    q2 = fmaf(x, x, q2);
                }
                char* at = to + (size_t)ch * 8 * kCutBlock;
                *reinterpret_cast<uint4*>(at + (u & 1) * 3072 + 2048 + (g * 32 + R) * 16) = make_uint4(q[0], q[1], q[2], q[3]);
                *reinterpret_cast<uint2*>(at + 6144 + (u & 1) * 512 + (g * 32 + R) * 8) = make_uint2(q[4], q[5]);
            }
        }
        __syncthreads();
    }
    float qh2 = (lane & 1) == 0 ? q2 : 0.0f, ql2 = (lane & 1) == 1 ? q2 : 0.0f;
    nrm = wave_sum(nrm);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo2 += __shfl_xor(lo2, o);
        over += __shfl_xor(over, o);
        qh2 += __shfl_xor(qh2, o);
        ql2 += __shfl_xor(ql2, o);
    }
    if (lane == 0) {
        const float back = power_of_two(-sw);
        const double full = -0.5 * nrm * (double)s;              // (a sample's chunks are scaled back as they are added up)
        hats[r] = k < K && full > (double)kSplitPadNorm ? (float)full : kSplitPadNorm;
        if (k < K) norms[k] = (float)(-0.5 * nrm);
        float up = (float)nrm;
        if ((double)up < nrm) up = nextafterf(up, INFINITY);
        most[wave][0] = k < K ? up : 0.0f;
        most[wave][1] = sqrtf(lo2) * back;
        most[wave][2] = sqrtf(qh2) * back;
        most[wave][3] = (sqrtf(ql2) + sqrtf(over)) * back;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int t = threadIdx.x;
        const float m = fmaxf(fmaxf(most[0][t], most[1][t]), fmaxf(most[2][t], most[3][t]));
        if (m > 0.0f) atomicMax(&scal[t == 0 ? 0 : kScalLo + t - 1], __float_as_uint(m));
    }
}

// ---------------------------------------------------------------------------------------------------------
// The samples' parts: a workgroup takes 32 rows, its wavefronts a chunk of 64 features at a time.  Lane (j, g) brings in eight features
// of each half unit of row j, centres them, scales them by the power of two that takes the largest of the row's chunk into [2^kTopBit,
// 2^(kTopBit + 1)), and cuts them: half-precision parts, and fp6 parts of what they leave over (lower lanes) and of them (upper lanes).
// ---------------------------------------------------------------------------------------------------------
// LIST: the rows of the re-decision list's entries, 32 of them to a block, once the search is through with the parts.  (The candidate pass
// gathered them from the blocks of the samples, where an entry's 224 bytes of a chunk lie in fourteen lines: 10^5 x 2000 uniform values on
// 1024 nodes, 202 us; cut again 21, and the pass over whole blocks 48.)
constexpr int kCutThreads = 512;

template <bool LIST>
__device__ __forceinline__ void cut_block(const BmuArgs& a, const WideArgs& p, int64_t block, int64_t total, float (*sums)[64][3])
{
    constexpr int WAVES = kCutThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, g = lane >> 5;
    const int64_t i = block * 32 + j;
    int64_t ic = i < total ? i : total - 1;
    if constexpr (LIST) ic = (int64_t)a.recheck[ic];
    const float* const row = a.X + (a.idx ? (int64_t)a.idx[ic] : ic) * a.ldx;
    char* const to = p.cut + (size_t)block * p.nch * kCutBlock;
    float* const scales = p.scales + (size_t)block * p.nch * 32;
    const float q_scale = g == 0 ? power_of_two(-3) : power_of_two(kTopBit - 2);
    float l2 = 0.0f, e2 = 0.0f, w2 = 0.0f;                  // lower lanes: of second parts; upper: of first parts
    for (int ch = wave; ch < p.nch; ch += WAVES) {
        float v[2][2][8];
        float most = 0.0f;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int f = ch * kCutChunk + 32 * u + 16 * kb + 8 * g + 4 * h, start = f < a.D - 4 ? f : a.D - 4;
                    const float4 x = load4(row + start), c = load4(a.centre + start);
                    float* o = &v[u][kb][4 * h];
                    // (windows shifted back at the end of the row: own elements only)
                    const int shift = f - start;
                    o[0] = shift <= 0 ? x.x - c.x : 0.0f;
                    o[1] = shift <= 1 ? x.y - c.y : 0.0f;
                    o[2] = shift <= 2 ? x.z - c.z : 0.0f;
                    o[3] = shift <= 3 ? x.w - c.w : 0.0f;
                    most = fmaxf(most, fmaxf(fmaxf(fabsf(o[0]), fabsf(o[1])), fmaxf(fabsf(o[2]), fabsf(o[3]))));
                }
        {
            unsigned int m = __float_as_uint(most), n = m;
            swap_words(m, n);
            most = fmaxf(__uint_as_float(m), __uint_as_float(n));
        }
        const int sx = scale_for(most);
        const float s = power_of_two(sx), fx = power_of_two(-sx);
        char* const at = to + (size_t)ch * kCutBlock;
        if (g == 0) scales[ch * 32 + j] = fx;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            unsigned int hi[8], lo[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const HalfPair h(v[u][t >> 2][2 * (t & 3)] * s, v[u][t >> 2][2 * (t & 3) + 1] * s);
                hi[t] = h.hi;
                lo[t] = h.lo;
            }
            *reinterpret_cast<uint4*>(at + u * 3072 + lane * 16) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *reinterpret_cast<uint4*>(at + u * 3072 + 1024 + lane * 16) = make_uint4(hi[4], hi[5], hi[6], hi[7]);
            uintx16 w;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                unsigned int m = lo[t], n = hi[t];
                swap_words(m, n);
                w[t] = m;
                w[8 + t] = n;
            }
            const uintx6 q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(__builtin_bit_cast(halfx32, w), q_scale);
            *reinterpret_cast<uint4*>(at + u * 3072 + 2048 + lane * 16) = make_uint4(q[0], q[1], q[2], q[3]);
            *reinterpret_cast<uint2*>(at + 6144 + u * 512 + lane * 8) = make_uint2(q[4], q[5]);
            if constexpr (LIST) continue;                       // (a listed sample has its norms)
            const uintx16 d = __builtin_bit_cast(uintx16, __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(q, q_scale));
            float s2 = 0.0f, r2 = 0.0f;
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const halfx2 o = __builtin_bit_cast(halfx2, (unsigned int)w[t]);
                const halfx2 r = o - __builtin_bit_cast(halfx2, (unsigned int)d[t]);
                s2 = __builtin_amdgcn_fdot2(o, o, s2, false);
                r2 = __builtin_amdgcn_fdot2(r, r, r2, false);
            }
            const float after = u == 0 ? 4.0f : 2.0f;           // MFMAs of the chunk from the unit's own on
            l2 = fmaf(s2 * fx, fx, l2);
            e2 = fmaf(r2 * fx, fx, e2);
            w2 = fmaf(after * after * s2 * fx, fx, w2);
        }
    }
    if constexpr (LIST) return;
    sums[wave][lane][0] = l2;
    sums[wave][lane][1] = e2;
    sums[wave][lane][2] = w2;
    __syncthreads();
    if (wave == 0) {
        for (int w = 1; w < WAVES; ++w) {
            l2 += sums[w][lane][0];
            e2 += sums[w][lane][1];
            w2 += sums[w][lane][2];
        }
        const float h2 = __shfl_xor(l2, 32), eh2 = __shfl_xor(e2, 32), ha2 = __shfl_xor(w2, 32);
        if (g == 0 && i < a.m)
            p.norm[i] = part_norms(a, l2, e2, h2, eh2, ha2, 4.0f, (float)(p.nch + 2), 1.0f, power_of_two(-(int)a.scal[kScalShift]));
    }
}

__global__ void __launch_bounds__(kCutThreads) bmu_cut_samples_kernel(const BmuArgs a, const WideArgs p)
{
    __shared__ float sums[kCutThreads / 64][64][3];
    cut_block<false>(a, p, blockIdx.x, a.m, sums);
}

__global__ void __launch_bounds__(kCutThreads) bmu_cut_listed_kernel(const BmuArgs a, const WideArgs p)
{
    const unsigned int count = a.scal[a.slot];
    if (count <= p.cand_min) return;
    for (int64_t block = blockIdx.x; block * 32 < (int64_t)count; block += gridDim.x) cut_block<true>(a, p, block, (int64_t)count, nullptr);
}

// ---------------------------------------------------------------------------------------------------------
// The tiles.  CAND: the samples are the entries of the re-decision list, and every node that reaches the entry's cut is
// appended to the sample's record (rare: an atomic each); the scores are those of the first pass bit for bit.
// ---------------------------------------------------------------------------------------------------------
template <bool CAND>
__device__ __forceinline__ void cut_tile(const BmuArgs& a, const WideArgs& p, int64_t tile, int split, int s_lo, int s_hi, int64_t total, char* lds)
{
    constexpr int AHEAD = kCutAhead, GROUPS = 2 * 6;
    static_assert(AHEAD == 2, "two places of each kind");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, g = lane >> 5;
    const int nch = p.nch;
    const int64_t wave0 = (tile * kCutWaves + wave) * 32;
    if (s_hi <= s_lo) return;                               // (whole workgroup)
    const int t_lo = s_lo >> 2, t_hi = (s_hi + 3) >> 2;
    float* const state = reinterpret_cast<float*>(lds + kCutStages * kCutStage) + wave * (kCutState * 64) + lane;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char*)lds);
    // this workgroup's stages of tile t: [first, end)
    auto first_of = [&](int t) { return t == t_lo ? s_lo & 3 : 0; };
    auto end_of = [&](int t) { return s_hi - 4 * t < 4 ? s_hi - 4 * t : 4; };
    // stage (t, ch, h) into its buffer: two 1 KB pieces a wavefront (of the fourteen the last two come twice, so that every wavefront has
    // as many loads under way)
    const unsigned lane16 = lane * 16, lane8 = 6144 + lane * 8;
    auto load_stage = [&](int t, int ch, int h, int buf) {
        const char* from = p.blob + (((size_t)t * nch + ch) * 4 + h) * kCutStage;
#pragma unroll
        for (int i = 0; i < kCutLoads; ++i) {
            int q = wave + kCutWaves * i;
            q = q < kCutStage / 1024 ? q : q - 2;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds0 + (unsigned)(buf * kCutStage + q * 1024)), "v"(lane16),
                         "s"(from + q * 1024)
                         : "memory", "m0");
        }
    };
    load_stage(t_lo, 0, s_lo & 3, 0);

    // ---- this wavefront's samples: lane (j, g) brings in eight features of each half unit of row j
    const int sw = (int)a.scal[kScalShift];
    const float back_w = power_of_two(-sw);
    const bool real = wave0 + j < total;
    int64_t entry = real ? wave0 + j : total - 1;
    float cut = NAN;                                        // no score compares >= NaN
    if constexpr (CAND) {
        if (real) cut = a.cutv[entry] * power_of_two(sw);
        entry = (int64_t)a.recheck[entry];
    }
    // parts of the chunk in hand and of the next one
    // (a block of 32 rows, the last one for wavefronts behind it)
    const int64_t blocks = (total + 31) / 32, block = wave0 / 32 < blocks ? wave0 / 32 : blocks - 1;
    const char* const parts = p.cut + (size_t)block * nch * kCutBlock;
    const float* const scales = p.scales + (size_t)block * nch * 32;
    const unsigned from8 = (unsigned)lane * 8, from4 = (unsigned)j * 4;
    struct Parts {
        uintx4 f[2][2];
        uintx6 q[2];
        float scale;
    };
    Parts now, then;
    auto load_parts = [&](Parts& x, int ch) {
        const char* at = parts + (size_t)ch * kCutBlock;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            x.f[u][0] = *reinterpret_cast<const uintx4*>(at + u * 3072 + lane16);
            x.f[u][1] = *reinterpret_cast<const uintx4*>(at + u * 3072 + 1024 + lane16);
            const uint4 q = *reinterpret_cast<const uint4*>(at + u * 3072 + 2048 + lane16);
            const uint2 r = *reinterpret_cast<const uint2*>(at + 6144 + u * 512 + from8);
            x.q[u][0] = q.x;
            x.q[u][1] = q.y;
            x.q[u][2] = q.z;
            x.q[u][3] = q.w;
            x.q[u][4] = r.x;
            x.q[u][5] = r.y;
        }
        x.scale = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(scales + ch * 32) + from4);
    };

    if constexpr (!CAND) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            state[(3 * c + 0) * 64] = -INFINITY;
            state[(3 * c + 1) * 64] = -INFINITY;
            state[(3 * c + 2) * 64] = 0.0f;
        }
    }
    floatx16 acc[8];
    // the scores of block b (as bmu_split_tile: two classes of rows, and, by nb's parity, two of blocks)
    auto fold = [&](const floatx16& v, int nb, int b) {
        if constexpr (CAND) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (v[r] >= cut) {
                    const int id = node_of_row(b * 32 + 8 * (r >> 2) + 4 * g + (r & 3), a.K);
                    uint32_t* rec = p.record + entry * kWRecord;
                    const unsigned at = atomicAdd(rec, 1u);
                    if (at < (unsigned)kWIds) reinterpret_cast<uint16_t*>(rec + 1)[at] = (uint16_t)id;
                }
        } else {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                float* st = state + (2 * (nb & 1) + c) * 3 * 64;
                float best = st[0], second = st[64];
                const float before = best;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r0 = 4 * q + c, r1 = r0 + 2;
                    const float v1 = __uint_as_float((__float_as_uint(v[r0]) & 0xfffffff8u) | (unsigned)(r0 >> 1));
                    const float v2 = __uint_as_float((__float_as_uint(v[r1]) & 0xfffffff8u) | (unsigned)(r1 >> 1));
                    const float mid = __builtin_amdgcn_fmed3f(best, v1, v2);
                    best = vmax3(best, v1, v2);
                    second = vmax(second, mid);
                }
                st[0] = best;
                st[64] = second;
                if (best > before) st[128] = __int_as_float(b);
            }
        }
    };

    // ---- fragments of the weights: a block's group 0 and 1 are its units' small products, then first parts, two MFMAs a unit
    uintx6 fq[2];
    uintx4 ff[2];
    auto read = [&](const char* base, int i) {
        const int w = i % 6;
        const char* at = base + i / 6 * kCutBlock;
        if (w < 2) {
            const uint4 t = *reinterpret_cast<const uint4*>(at + lane16 + w * 3072 + 2048);
            const uint2 r = *reinterpret_cast<const uint2*>(at + lane8 + w * 512);
            fq[w] = uintx6{t.x, t.y, t.z, t.w, r.x, r.y};
        } else {
            ff[w & 1] = *reinterpret_cast<const uintx4*>(at + lane16 + ((w - 2) >> 1) * 3072 + ((w - 2) & 1) * 1024);
        }
    };
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int scale_a = g == 0 ? 127 + kTopBit - 2 : 127 - 3, scale_b = g == 0 ? 127 - 3 : 127 + kTopBit - 2;
    auto follow = [&](int& t, int& ch, int& h) {            // the stage after (t, ch, h)
        if (++h >= end_of(t)) {
            if (++ch == nch) {
                ch = 0;
                ++t;
            }
            h = first_of(t);
        }
    };
    int tn = t_lo, cn = 0, hn = s_lo & 3;                   // the stage that is requested next
    int buf = 0;
    // One stage of NST: two blocks, acc[2 h] and the next; ch1: the next chunk.  At its barrier the next stage has to be there.  Of the loads
    // behind that one two, of the stage after it, may still be under way, and from the chunk's second stage on also those of the
    // next chunk's parts, requested at its first one (nine, of which seven are counted on); where no stage is left to be requested, none.
    // In the chunk's last stage everything has to be there, the parts among it.
    auto stage = [&](auto which, auto of, int ch1) {
        constexpr int h = decltype(which)::value, NST = decltype(of)::value;
        const char* base = lds + buf * kCutStage;
        const int buf1 = (buf + 1) & 3;
        const char* next = lds + buf1 * kCutStage;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            floatx16 part;
#pragma unroll
            for (int w = 0; w < 6; ++w) {
                const int i = 6 * nb + w;
                if (w < 2) {
                    part = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(fq[w]), fp6_operand(now.q[w]), w == 0 ? zero16 : part, 2, 2, 0,
                                                                           scale_a, 0, scale_b);
                } else {
                    part = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, ff[w & 1]), __builtin_bit_cast(halfx8, now.f[(w - 2) >> 1][(w - 2) & 1]), part, 0, 0, 0);
                }
                if (i + AHEAD < GROUPS) {
                    read(base, i + AHEAD);
                } else if (i + AHEAD == GROUPS) {
                    // (everything of this stage has been read: the barrier gives its place away)
                    static_assert(kCutLoads == 2, "the counts");
                    const bool more = tn < t_hi;
                    if (h == NST - 1 || !more) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else if (h == 0) asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    else asm volatile("s_waitcnt vmcnt(9) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    if constexpr (h == NST - 1) {
                        // (the compiler waits for the parts where they are first touched, and knows none of the other loads: here)
#pragma unroll
                        for (int u = 0; u < 2; ++u) asm volatile("" : "+v"(then.q[u]), "+v"(then.f[u][0]), "+v"(then.f[u][1]));
                        asm volatile("" : "+v"(then.scale));
                    }
                    if (more) {
                        load_stage(tn, cn, hn, (buf + 3) & 3);
                        follow(tn, cn, hn);
                    }
                    if constexpr (h == 0 && NST > 1) load_parts(then, ch1);
                    read(next, 0);
                } else {
                    read(next, i + AHEAD - GROUPS);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[2 * h + nb][r] = fmaf(part[r], now.scale, acc[2 * h + nb][r]);
            asm volatile("" : "+v"(acc[2 * h + nb]));           // (here, not behind the branches that follow: the parts' registers)
        }
        buf = buf1;
    };
    // NST stages of node tile t, from stage h0 on
    auto node_tile = [&](auto of, int t, int h0) {
        constexpr int NST = decltype(of)::value;
        const float4* n4 = reinterpret_cast<const float4*>(p.hats + (size_t)t * kCutTile + h0 * 64) + g;
#pragma unroll
        for (int nb = 0; nb < 2 * NST; ++nb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 n = n4[nb * 8 + 2 * q];
                acc[nb][4 * q + 0] = n.x;
                acc[nb][4 * q + 1] = n.y;
                acc[nb][4 * q + 2] = n.z;
                acc[nb][4 * q + 3] = n.w;
            }
#pragma unroll
        for (int nb = 0; nb < 2 * NST; ++nb) asm volatile("" : "+v"(acc[nb]));      // (waited for here, not in every chunk)
        for (int ch = 0; ch < nch; ++ch) {
            const int ch1 = ch + 1 < nch ? ch + 1 : 0;          // (behind the last chunk of all it is loaded for nothing)
            if constexpr (NST == 1) load_parts(then, ch1);
            stage(std::integral_constant<int, 0>{}, of, ch1);
            if constexpr (NST > 1) stage(std::integral_constant<int, 1>{}, of, ch1);
            if constexpr (NST > 2) stage(std::integral_constant<int, 2>{}, of, ch1);
            if constexpr (NST > 3) stage(std::integral_constant<int, 3>{}, of, ch1);
            now = then;
        }
#pragma unroll
        for (int nb = 0; nb < 2 * NST; ++nb)
            if (t * kCutTile + h0 * 64 + nb * 32 < a.K) fold(acc[nb], nb, 8 * t + 2 * h0 + nb);
    };

    load_parts(now, 0);
    follow(tn, cn, hn);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
    for (int b = 1; b < kCutStages - 1; ++b)
        if (tn < t_hi) {
            load_stage(tn, cn, hn, b);
            follow(tn, cn, hn);
        }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read(lds, i);

    // (a piece of a node tile, or whole tiles and, at the end of the map, a piece)
    const int whole = (s_lo & 3) != 0 ? t_lo : s_hi >> 2;
    for (int t = t_lo; t < whole; ++t) node_tile(std::integral_constant<int, 4>{}, t, 0);
    if (whole < t_hi) {
        const int h0 = first_of(whole), nst = end_of(whole) - h0;
        if (nst == 1) node_tile(std::integral_constant<int, 1>{}, whole, h0);
        else node_tile(std::integral_constant<int, 2>{}, whole, h0);
    }
    if constexpr (CAND) return;

    // ---- the sample's eight class winners of this workgroup: the four best with their ids, and the highest of all others
    float won[8];
    int where[8];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        won[c] = state[3 * c * 64];
        where[c] = __float_as_int(state[(3 * c + 2) * 64]);
        won[4 + c] = __shfl_xor(won[c], 32);
        where[4 + c] = __shfl_xor(where[c], 32);
    }
    float others = fmaxf(fmaxf(state[64], state[4 * 64]), fmaxf(state[7 * 64], state[10 * 64]));
    others = fmaxf(others, __shfl_xor(others, 32));
    if (g == 0 && real) write_winners(a, p, split, entry, won, where, others, back_w);
}

// what workgroup blockIdx.x does
struct CutUnit {
    int64_t tile;
    int split, per;
};
__device__ __forceinline__ CutUnit cut_unit(const WideArgs& p)
{
    // (at most 2^24 rows a pass and 16 pieces: 32 bits)
    const unsigned first = (unsigned)((p.tail_tile + 7) / 8 * 8) * (unsigned)p.splits;
    const bool tail = blockIdx.x >= first;
    const unsigned splits = (unsigned)(tail ? p.tail_splits : p.splits), b = blockIdx.x - (tail ? first : 0u), within = b % (8u * splits);
    const int tile = __builtin_amdgcn_readfirstlane((int)(b / (8u * splits) * 8u + within % 8u)), split = __builtin_amdgcn_readfirstlane((int)(within / 8u));
    // (numbers behind the last tile, of either kind, are nobody's)
    return {tail ? p.tail_tile + tile : tile < p.tail_tile ? (int64_t)tile : (int64_t)1 << 40, split, tail ? p.tail_per : p.per_split};
}

// The splits of a sample tile get workgroup numbers 8 apart: they run on the same XCD at about the same time, and its L2 serves the
// parts to all but the first.  The sample tiles of the last, partial round are split further (tail).
__global__ void __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_cut_split_kernel(const BmuArgs a, const WideArgs p)
{
    extern __shared__ float4 cut_lds[];
    const CutUnit u = cut_unit(p);
    if (u.tile * kCutRows >= a.m) return;
    const int stages = cut_stages(a.K), s_lo = u.split * u.per, s_hi = s_lo + u.per < stages ? s_lo + u.per : stages;
    cut_tile<false>(a, p, u.tile, u.split, s_lo, s_hi, a.m, reinterpret_cast<char*>(cut_lds));
}

// A fixed grid walks the (tile of the list, piece of the map) units; a short list takes smaller pieces, so that it still spreads over the chip.
__global__ void __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_cut_split_cand_kernel(const BmuArgs a, const WideArgs p)
{
    extern __shared__ float4 cut_lds[];
    const unsigned int count = a.scal[a.slot];
    if (count <= p.cand_min) return;
    const unsigned stages = cut_stages(a.K), tiles = (count + kCutRows - 1) / kCutRows;       // (at most 2^24 rows and 65536 nodes a pass)
    // (rounds times a piece's stages and seven, as bmu_cut_plan)
    unsigned per = 4, least = 0xffffffffu;
    for (unsigned n = 4; n > 0; n >>= 1) {
        const unsigned time = (tiles * ((stages + n - 1) / n) + gridDim.x - 1) / gridDim.x * (n + 7);
        if (time < least) {
            least = time;
            per = n;
        }
    }
    const unsigned pieces = (stages + per - 1) / per;
    for (unsigned u = blockIdx.x; u < tiles * pieces; u += gridDim.x) {
        const int tile = __builtin_amdgcn_readfirstlane((int)(u / pieces)), piece = __builtin_amdgcn_readfirstlane((int)(u % pieces));
        const int s_lo = piece * (int)per, s_hi = s_lo + (int)per < (int)stages ? s_lo + (int)per : (int)stages;
        cut_tile<true>(a, p, tile, 0, s_lo, s_hi, (int64_t)count, reinterpret_cast<char*>(cut_lds));
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------
size_t bmu_cut_blob_bytes(int32_t K, int32_t D)
{
    return cut_blob(K, D) + ((size_t)cut_rows(K) + (size_t)K + ((size_t)D + 63) / 64) * sizeof(float);
}

static float* cut_hats(const BmuPrep& prep, int32_t K, int32_t D) { return (float*)((char*)prep.stage16 + cut_blob(K, D)); }

float* bmu_cut_spread(const BmuPrep& prep, int32_t K, int32_t D) { return cut_hats(prep, K, D) + cut_rows(K) + K; }

int bmu_cut_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small)
{
    const int nch = (D + kCutChunk - 1) / kCutChunk;
    float* hats = cut_hats(prep, K, D);
    const int64_t rows = cut_rows(K), groups = rows / 4 + ((int64_t)D * prep.kpad + 255) / 256;
    hipLaunchKernelGGL(bmu_cut_prep_kernel, dim3((unsigned)groups), dim3(256), 0, ctx->stream, W, K, D, prep.kpad, (int)rows, nch,
                       prep.centre, bmu_cut_spread(prep, K, D), (char*)prep.stage16, hats, hats + rows, prep.wt, prep.scal, qe, small);
    return check_hip(ctx, hipGetLastError(), "bmu (rows cut beforehand) preparation launch");
}

size_t bmu_cut_scales_bytes(int32_t D, int64_t m) { return ((size_t)m + 31) / 32 * (((size_t)D + kCutChunk - 1) / kCutChunk) * 32 * sizeof(float); }
size_t bmu_cut_parts_bytes(int32_t D, int64_t m) { return ((size_t)m + 31) / 32 * (((size_t)D + kCutChunk - 1) / kCutChunk) * kCutBlock; }

// The parts take 3.6 bytes a value: passes of as many rows as a gigabyte holds.  (Passes that stay in the 256 MB cache beside the memory
// don't make the cut faster, 10^5 x 2000: 360 us in passes of 192 MB instead of 331, and the short lists of every pass cost another
// 100 us each.)
int64_t bmu_cut_pass_rows(int32_t D)
{
    const int64_t rows = ((int64_t)1 << 30) / (((int64_t)D + kCutChunk - 1) / kCutChunk * (kCutBlock / 32 + 4)) / kCutRows * kCutRows;
    return rows < kCutRows ? kCutRows : rows;
}

// What workgroups take: pieces of the map's stages, a unit one piece at a time.  The time goes with the rounds, times the stages of a piece and
// about seven more (10^5 x 2000: 93 us a round of one stage, 126 of four).  Whole rounds of sample tiles in pieces of whole node tiles, by
// preference of one: four and more pieces of a sample tile share its parts in an XCD's L2, and eight sample tiles the weights' (10^5 x 2000 on
// 1024 nodes in pieces of four node tiles: 823 us instead of 727).  What is left over goes into smaller pieces, down to a stage, where an XCD's
// eighth of the units then holds its eighth of the sample tiles: 10^5 x 2000 on 1024 nodes 1092 -> 1059 us, 22,526 x 951 on 1024 137 -> 125, 11,414 x
// 914 on 530 72 -> 59; with two rounds of them 10,618 x 916 on 729 72 -> 88.  Behind whole rounds only where sample tiles have no short last piece or
// four pieces and more: units that are through with short pieces take up the rest as it is (43,989 x 444 on 576 nodes 90 us, 93 in smaller pieces).
void bmu_cut_plan(WideArgs& p, const BmuPrep& prep, int64_t m, int32_t K, int32_t D, int units)
{
    p.nch = (D + kCutChunk - 1) / kCutChunk;
    p.hats = cut_hats(prep, K, D);
    p.norms = p.hats + cut_rows(K);
    const int64_t tiles = (m + kCutRows - 1) / kCutRows;
    const int steps = cut_stages(K), whole = 4;
    auto cost_of = [&](int64_t n, int per) { return (double)((n * ((steps + per - 1) / per) + units - 1) / units) * ((double)per + 7.0); };
    double best = 0.0;
    for (int s = 1; s <= 16 && (s == 1 || s <= (steps + whole - 1) / whole); ++s) {
        const int per = ((steps + s - 1) / s + whole - 1) / whole * whole, pieces = (steps + per - 1) / per;
        if (pieces < 4 && per > whole) continue;
        int64_t first = tiles * pieces / units * units / pieces / 8 * 8;          // (the numbering goes by eight tiles)
        if (tiles * pieces % units == 0) first = tiles;
        int tail = per;
        for (int t = per - whole; t >= 1 && first < tiles; t = t > whole ? t - whole : t / 2)        // (none where a piece is a node tile)
            if ((steps + t - 1) / t <= 16 && cost_of(tiles - first, t) < cost_of(tiles - first, tail) * 0.98) tail = t;
        const double cost = (first > 0 ? cost_of(first, per) : 0.0) + (first < tiles ? cost_of(tiles - first, tail) : 0.0);
        if (best > 0.0 && !(cost < best * 0.98)) continue;
        best = cost;
        p.per_split = per;
        p.splits = pieces;
        p.tail_tile = first;
        p.tail_per = tail;
    }
    const int64_t first = p.tail_tile, last = tiles - first;
    if (p.per_split == whole && last > 0 && (first == 0 || p.splits >= 4 || steps % whole == 0)) {
        const int64_t eighth = units < 8 ? 1 : units / 8;                         // (every eighth workgroup runs on the same XCD)
        auto cost_on_one = [&](int per) { return (double)(((last + 7) / 8 * ((steps + per - 1) / per) + eighth - 1) / eighth) * ((double)per + 7.0); };
        for (int t = whole / 2; t >= 1; t /= 2)
            if ((steps + t - 1) / t <= 16 && cost_on_one(t) < cost_on_one(p.tail_per) * 0.98) p.tail_per = t;
    }
    p.tail_row = first * kCutRows < m ? first * kCutRows : m;
    p.tail_splits = (steps + p.tail_per - 1) / p.tail_per;
    p.grid = (first + 7) / 8 * 8 * p.splits + (last + 7) / 8 * 8 * p.tail_splits;
}

int bmu_cut_launch(som_ctx* ctx, const BmuArgs& a, const WideArgs& p, bool cand)
{
    if (cand) {
        const int64_t blocks = (a.m + 31) / 32;
        hipLaunchKernelGGL(bmu_cut_listed_kernel, dim3((unsigned)(blocks < 1024 ? blocks : 1024)), dim3(kCutThreads), 0, ctx->stream, a, p);
        if (int rc = check_hip(ctx, hipGetLastError(), "bmu (rows cut beforehand) list cut launch")) return rc;
        hipLaunchKernelGGL(bmu_cut_split_cand_kernel, dim3(256), dim3(kTileThreads), kCutLds, ctx->stream, a, p);
        return check_hip(ctx, hipGetLastError(), "bmu (rows cut beforehand) candidate launch");
    }
    static bool attr_set_dev[kMaxDevices] = {};
    const void* kernels[] = {reinterpret_cast<const void*>(bmu_cut_split_kernel), reinterpret_cast<const void*>(bmu_cut_split_cand_kernel)};
    if (int rc = wide_raise_lds(ctx, attr_set_dev, kernels, kCutLds)) return rc;
    hipLaunchKernelGGL(bmu_cut_samples_kernel, dim3((unsigned)((a.m + 31) / 32)), dim3(kCutThreads), 0, ctx->stream, a, p);
    if (int rc = check_hip(ctx, hipGetLastError(), "bmu (rows cut beforehand) cut launch")) return rc;
    hipLaunchKernelGGL(bmu_cut_split_kernel, dim3((unsigned)p.grid), dim3(kTileThreads), kCutLds, ctx->stream, a, p);
    return check_hip(ctx, hipGetLastError(), "bmu (rows cut beforehand) search launch");
}

} // namespace som
