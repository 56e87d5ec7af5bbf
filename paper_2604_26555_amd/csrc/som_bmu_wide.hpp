// What the searches for more than 64 features share (som_bmu_wide.hip, som_bmu_held.hip, som_bmu_cut.hip): a pass's workspace and its join.
#pragma once

#include "som_bmu_common.hpp"

namespace som {

constexpr int kWIds = 14;                         // candidate ids of a record: 4 bytes count, fourteen 16-bit ids
constexpr int kWRecord = 8;                       // 32-bit words of a record
constexpr int kHeldFeatures = 256;                // most features of a row that the wavefronts hold (som_bmu_held.hip)

struct WideArgs {
    const char* blob;        // weights' parts
    const float* hats;       // -|w|^2 / 2 at the weights' scale, in the order of the rows
    const float* norms;      // [K] -|w|^2 / 2
    int nch, tiles;          // chunks of a row; node tiles (som_bmu_wide.hip)
    int splits, per_split;   // workgroups that share a sample tile, steps (node tiles, stages of 64 nodes or blocks of 32) of each
    int tail_splits, tail_per;                   // the same of the sample tiles from tail_tile, and the rows from tail_row, on
    int64_t tail_tile, tail_row, grid;
    int64_t rows;            // m of the pass
    float4* best;            // [result] best, second best class winner, highest of all but the best four; id of the best (bits)
    uint4* next;             // [result] third and fourth (bits); 16-bit ids of the second and third, of the fourth
    float4* norm;            // [m] |x|, and what a score errs by at most: y |w| + z + rounding of |w|^2 / 2 (bf16 parts: |x|^2, weighted |x|^2, |x - hi|^2)
    uint32_t* record;        // [m][kWRecord] candidates of the listed samples
    char* cut;               // the samples' parts, [block of 32][chunk], as a block of the weights; and the scales that take them back, [32] each
    float* scales;
    uint32_t cand_min;       // lists up to this length go to the all-nodes pass at once

    // all sample tiles alike
    void set_splits(int64_t m, int n, int per, int64_t groups)
    {
        splits = tail_splits = n;
        per_split = tail_per = per;
        tail_tile = tail_row = m;
        grid = groups;
    }
    // Where the workgroup with number `split` of a sample leaves its winners: [splits][tail_row], then [tail_splits][rows - tail_row].  (The tail has up
    // to sixteen splits and few rows: 32 bytes for every row and each of them would be most of a pass's memory.)
    __host__ __device__ size_t result(int split, int64_t i) const
    {
        return i < tail_row ? (size_t)split * tail_row + i : (size_t)splits * tail_row + (size_t)split * (rows - tail_row) + (i - tail_row);
    }
    size_t results() const { return (size_t)splits * tail_row + (size_t)tail_splits * (rows - tail_row); }
};

typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx32 __attribute__((ext_vector_type(32)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned int uintx6 __attribute__((ext_vector_type(6)));
typedef unsigned int uintx8 __attribute__((ext_vector_type(8)));
typedef unsigned int uintx16 __attribute__((ext_vector_type(16)));
typedef int intx8 __attribute__((ext_vector_type(8)));

constexpr int kTopBit = 11;      // the largest element is scaled into [2^11, 2^12): what its half-precision part leaves over is below 1

__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }

// the scale exponent that takes `most`, the largest magnitude, into [2^kTopBit, 2^(kTopBit + 1))
__device__ __forceinline__ int scale_for(float most)
{
    const int e = kTopBit + 127 - (int)(__float_as_uint(most) >> 23 & 255u);
    return e < -90 ? -90 : e > 90 ? 90 : e;
}

// two values' half-precision parts and those of what they leave over
struct HalfPair {
    unsigned int hi, lo;
    __device__ __forceinline__ HalfPair(float x0, float x1)
    {
        const floatx2 x = {x0, x1};
        const halfx2 h = __builtin_convertvector(x, halfx2);
        halfx2 l;
        l[0] = (_Float16)fmaf((float)h[0], -1.0f, x0);
        l[1] = (_Float16)fmaf((float)h[1], -1.0f, x1);
        hi = __builtin_bit_cast(unsigned int, h);
        lo = __builtin_bit_cast(unsigned int, l);
    }
};

// the two halves of a wavefront trade: a keeps its lower half's and takes b's, b takes a's upper half's and keeps its own
__device__ __forceinline__ void swap_words(unsigned int& a, unsigned int& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// thirty-two fp6 values as the MFMA's builtin takes them (of the eight words six are read)
__device__ __forceinline__ intx8 fp6_operand(const uintx6& v)
{
    return __builtin_bit_cast(intx8, (uintx8)__builtin_shufflevector(v, v, 0, 1, 2, 3, 4, 5, -1, -1));
}

// What a score of a sample errs by, for WideArgs::norm, from the squares of its second parts and of what their rounding to fp6 leaves
// over (l2, e2), of its first parts likewise (h2, eh2), and of the first parts weighted by the MFMAs that follow (ha2); back: the factor
// that takes their roots to the values as given; back_w: the weights' 2^-(scale).
// (1) What the cuts drop: with x = xh + xl and its fp6 parts qh and ql, w likewise, |xl - ql| |w| + |ql| |wh - qh_w| + |xh - qh| |wl| +
// |qh| |wl - ql_w| + |xl| |wl|, from norms that were formed (the weights' are the largest over the nodes).  (2) The pipe's
// accumulation, as in bmu_split_tile: an MFMA of half-precision products is charged sixteen units of its accumulator and products,
// those of fp6 products, sixty-four terms each, hold small numbers only (cross: how many there are, and two).  (3) Ten units for the
// centrings and the norm, and one for each of `adds` additions of partial sums.  (A second part is rounded to half precision
// before it goes to fp6, and a subnormal part costs what 2^-14 would: 2^-25 of the largest.)
__device__ __forceinline__ float4 part_norms(const BmuArgs& a, float l2, float e2, float h2, float eh2, float ha2, float cross, float adds, float back,
                                             float back_w)
{
    constexpr float unit = 5.9604645e-08f;
    auto root = [&](float x) { return __builtin_amdgcn_sqrtf(x + kSquaresFloor) * (1.001f * back); };
    const float nh = root(h2), nx = nh + root(l2) * 1.001f, nl = root(l2) * 1.001f + nx * 1.0e-9f;
    const float ql = root(e2) + nl * 4.9e-4f + nx * 1.0e-9f, qh = root(eh2);
    const float lo_w = __uint_as_float(a.scal[kScalLo]) * 1.001f, qh_w = __uint_as_float(a.scal[kScalLo + 1]) * 1.001f,
                ql_w = __uint_as_float(a.scal[kScalLo + 2]) * 1.001f;
    const float small = 80.0f * unit * cross;
    const float err_w = ql * 1.001f + root(ha2) * (16.3f * unit) + nl * small + nx * ((10.0f + adds) * unit);
    const float err_0 = 1.001f * ((nl + ql) * qh_w + qh * lo_w + (nh + qh) * ql_w + nl * lo_w) + nx * (lo_w * small + back_w * 1.0e-7f);
    return make_float4(nx, err_w, err_0, 0.0f);
}

// A sample's class winners of a workgroup: the four best with their ids, and the highest of all others.  (Whoever reaches the sample's cut and is
// none of the four sends it through the tiles again: 10^5 x 2000 uniform values on 1024 nodes, 436 us with two kept, 204 with four.)
struct BestFour {
    float v[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, others;
    int id[4] = {0, 0, 0, 0};
    __device__ __forceinline__ explicit BestFour(float others_) : others(others_) {}
    __device__ __forceinline__ void add(float x, int row)
    {
        others = fmaxf(others, fminf(v[3], x));
        bool above[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) above[t] = x > v[t];
#pragma unroll
        for (int t = 3; t > 0; --t) {
            id[t] = above[t - 1] ? id[t - 1] : above[t] ? row : id[t];
            v[t] = __builtin_amdgcn_fmed3f(x, v[t - 1], v[t]);
        }
        id[0] = above[0] ? row : id[0];
        v[0] = fmaxf(v[0], x);
    }
    __device__ __forceinline__ void write(const WideArgs& p, int split, int64_t i, float back)
    {
        const size_t at = p.result(split, i);
        p.best[at] = make_float4(v[0] * back, v[1] * back, others * back, __int_as_float(id[0]));
        p.next[at] = make_uint4(__float_as_uint(v[2] * back), __float_as_uint(v[3] * back), (unsigned)id[1] & 0xffffu | (unsigned)id[2] << 16, (unsigned)id[3] & 0xffffu);
    }
};

// the same of eight class winners as held and cut rows leave them (places 4 and up: rows of the upper lane half; their blocks of 32 rows in `where`)
__device__ __forceinline__ void write_winners(const BmuArgs& a, const WideArgs& p, int split, int64_t i, const float (&won)[8], const int (&where)[8],
                                              float others, float back)
{
    BestFour b(others);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int r = 2 * (int)(__float_as_uint(won[q]) & 7u) + (q & 1);
        b.add(won[q], where[q] * 32 + 8 * (r >> 2) + 4 * (q >> 2) + (r & 3));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) b.id[t] = node_of_row(b.id[t], a.K);
    b.write(p, split, i, back);
}

// 64 lanes x 16 bytes, from the lanes' own addresses to 1 KB of LDS at offset lds (below 64 KB); counted by vmcnt
__device__ __forceinline__ void lds_load16(const void* from, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(from) : "memory", "m0");
}

// Which search rows of more than 64 features take: held in the wavefronts' registers (som_bmu_held.hip) where they fit; wider ones are cut once
// beforehand (som_bmu_cut.hip), except on small maps, where that pass over memory costs more than the shorter products give back
// (som_bmu_wide.hip).  Up to 512 nodes, two tiles of nodes, the tile also stays ahead where the rows are many and fill its rounds (bmu_wide_form).
// Whole search, 10^5 rows, cut beforehand against the tile: 600 features 311 us and 299 on 320 nodes, 309 and 289 on 361,
// 423 and 531 on 1024; 2000 features 915 and 955, 902 and 997, 1172 and 1707; on 256 nodes 787 and 685.
enum WideForm { kWideTile, kWideHeld, kWideCut };
constexpr int kCutNodes = 320;                    // most nodes that the tile always takes,
constexpr int kCutNodesMany = 512;                // and most that it takes for many rows

// spread: where the centre's kernel leaves the largest |w - centre| of every 64 features (null: not asked for)
float* bmu_wide_spread(const BmuPrep& prep, int32_t K, int32_t D);
int wide_raise_lds(som_ctx* ctx, bool* done, const void* const (&kernels)[2], size_t bytes);

size_t bmu_held_blob_bytes(int32_t kpad, int32_t D);
float* bmu_held_spread(const BmuPrep& prep, int32_t D);
int bmu_held_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small);
void bmu_held_plan(WideArgs& p, const BmuPrep& prep, int64_t m, int32_t K, int32_t D, int units);
int bmu_held_launch(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, const WideArgs& p, bool cand);

size_t bmu_cut_blob_bytes(int32_t K, int32_t D);
float* bmu_cut_spread(const BmuPrep& prep, int32_t K, int32_t D);
size_t bmu_cut_scales_bytes(int32_t D, int64_t m);
size_t bmu_cut_parts_bytes(int32_t D, int64_t m);
int64_t bmu_cut_pass_rows(int32_t D);
int bmu_cut_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small);
void bmu_cut_plan(WideArgs& p, const BmuPrep& prep, int64_t m, int32_t K, int32_t D, int units);
int bmu_cut_launch(som_ctx* ctx, const BmuArgs& a, const WideArgs& p, bool cand);

} // namespace som
