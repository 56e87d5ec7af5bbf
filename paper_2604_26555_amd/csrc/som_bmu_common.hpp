// Device helpers shared by the best-matching-unit kernels (som_bmu.hip and the three wide forms).
#pragma once

#include "som_internal.hpp"

#include <hip/amd_detail/amd_hip_unsafe_atomics.h>

namespace som {

typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

constexpr int kScalLo = 8;        // scal[8], scal[9]: bits of the largest |w - hi|^2 and |w - hi - lo|^2 (split search); three figures of
                                  // som_bmu_held.hip
constexpr int kScalShift = 11;    // scal[11]: the weights' scale there

// Added to the sums of squares that enter a bound before their root is taken: v_sqrt_f32 returns zero for a subnormal number, which
// would take up to 2^-63 from a norm.  The sums themselves keep subnormal squares, those by v_dot2c_f32_bf16 (square2) as
// well as those by fma (seen for squares and sums of 2^-112 to 2^-142), and what is lost below that, 2^-149 a square, is
// covered too.
constexpr float kSquaresFloor = 1e-37f;

constexpr float kSplitPadNorm = -3.0e38f;     // padding nodes of the split search: finite, so that position bits cannot make a NaN

// Sum of distances and squared distances of a workgroup's samples -> one of kQeSlots partial-sum slots.  Every
// wavefront adding to the same two words would serialise tens of thousands of atomics on one address; one pair
// per workgroup spread over 256 slots does not show in the kernel time.  Called by all threads of the workgroup.
// near: the split searches also count this lane's near ties, into kQeSlots further slots (counts are whole numbers: exact).
__device__ __forceinline__ void group_qe_add(double* __restrict__ part, double qs, double qs2, int near = 0)
{
    __shared__ double wsum[16][2];
    __shared__ int wnear[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) near += __shfl_xor(near, o);
    qs = wave_sum(qs);
    qs2 = wave_sum(qs2);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        wsum[wave][0] = qs;
        wsum[wave][1] = qs2;
        wnear[wave] = near;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t0 = 0.0, t1 = 0.0;
        int t2 = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            t0 += wsum[w][0];
            t1 += wsum[w][1];
            t2 += wnear[w];
        }
        if (t2 != 0) unsafeAtomicAdd(&part[2 * kQeSlots + (blockIdx.x & (kQeSlots - 1))], (double)t2);
        if (t0 != 0.0 || t1 != 0.0) {
            const int slot = blockIdx.x & (kQeSlots - 1);
            unsafeAtomicAdd(&part[2 * slot], t0);
            unsafeAtomicAdd(&part[2 * slot + 1], t1);
        }
    }
}

// Append sample i (and its score cut) to the re-decision list for every lane with `push` set: one atomic per wavefront (the list
// length is a single word; one atomic per listed sample serialises on it when a tenth of all samples is listed).
// Called in converged control flow by all lanes of the wavefront.
__device__ __forceinline__ void list_push(unsigned int* __restrict__ counter, uint32_t* __restrict__ list,
                                          float* __restrict__ cutv, bool push, int64_t i, float cut)
{
    const unsigned long long mask = __ballot(push);
    if (mask == 0ull) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((long long)mask) - 1;
    unsigned int base = 0u;
    if (lane == leader) base = atomicAdd(counter, (unsigned int)__popcll(mask));
    base = __shfl(base, leader);
    const unsigned int below = __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
    if (push) {
        list[base + below] = (uint32_t)i;
        if (cutv) cutv[base + below] = cut;     // scores at or above this value may belong to the true winner
    }
}

// A sample whose few candidates the search already knows (kPairs; their ids are in a.pairs) goes on the pair list, which
// grows down from the end of the same array.
constexpr float kNotListed = __builtin_nanf("");
constexpr float kPairs = __builtin_inff();

// The cut of a listed sample.  A row that holds no number, or whose scores overflow, has none and reads like one of the two
// marks above: any node may be its winner.
__device__ __forceinline__ float list_cut(float cut) { return fabsf(cut) < INFINITY ? cut : -INFINITY; }

// sixteen bytes from a 4-byte aligned address in one load (global memory needs no more than dword alignment)
__device__ __forceinline__ float4 load4(const float* p)
{
    float4 v;
    __builtin_memcpy(&v, p, sizeof(v));
    return v;
}

// 64 lanes x 16 bytes, from `base` (the same for all lanes) + the lane's offset to 1 KB of LDS at offset lds (below 64 KB); counted by vmcnt
__device__ __forceinline__ void lds_load16(const char* base, unsigned offset, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}

// plain v_max_f32: the scores are never signalling NaNs worth quieting, and every VALU instruction here is paid
// for in matrix time (float32 MFMA and the vector ALU share the same lanes)
__device__ __forceinline__ float vmax(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// plain v_max3_f32, for the same reason
__device__ __forceinline__ float vmax3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Two floats and their two bf16 parts: one conversion per pair and part (element by element the compiler takes three), a shift or a
// mask back to float, exact differences.
struct SplitPair {
    uint32_t hi, lo;
    float left0, left1;

    __device__ __forceinline__ SplitPair(float v0, float v1)
    {
        hi = pack(v0, v1);
        left0 = v0 - first(hi);
        left1 = v1 - second(hi);
        lo = pack(left0, left1);
    }
    static __device__ __forceinline__ uint32_t pack(float v0, float v1)
    {
        const floatx2 v = {v0, v1};
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    }
    static __device__ __forceinline__ float first(uint32_t p) { return __uint_as_float(p << 16); }
    static __device__ __forceinline__ float second(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }
    // sum + the squares of what both parts leave over
    __device__ __forceinline__ float rest2(float sum) const
    {
        const float r0 = left0 - first(lo), r1 = left1 - second(lo);
        return fmaf(r1, r1, fmaf(r0, r0, sum));
    }
};

// sum + the squares of a pair of parts (v_dot2c_f32_bf16: for norms that enter bounds with a factor to spare and kSquaresFloor)
__device__ __forceinline__ float square2(uint32_t p, float sum)
{
    const bf16x2 v = __builtin_bit_cast(bf16x2, p);
    return __builtin_amdgcn_fdot2_f32_bf16(v, v, sum, false);
}

__device__ __forceinline__ void split8(const float (&v)[8], bf16x8& hi, bf16x8& lo)
{
    uint4 h, l;
    uint32_t* hp = &h.x;
    uint32_t* lp = &l.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const SplitPair p(v[2 * i], v[2 * i + 1]);
        hp[i] = p.hi;
        lp[i] = p.lo;
    }
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

// the same with the squares of the first parts, of the second parts and of what both leave over
__device__ __forceinline__ void split8(const float (&v)[8], bf16x8& hi, bf16x8& lo, float& hi2, float& lo2, float& rest2)
{
    uint4 h, l;
    uint32_t* hp = &h.x;
    uint32_t* lp = &l.x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const SplitPair p(v[2 * i], v[2 * i + 1]);
        hp[i] = p.hi;
        lp[i] = p.lo;
        hi2 = square2(p.hi, hi2);
        lo2 = square2(p.lo, lo2);
        rest2 = p.rest2(rest2);
    }
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

// ---------------------------------------------------------------------------------------------------------
// Which node a row of the stages holds.  The search keeps its winners by class of rows (bits 0, 2 and 5 of the row: bmu_split_tile), and
// a near tie within one class costs a pass of its own, so nodes that come close should fall into different classes: the rows of a
// whole stage of 128 are ordered such that those three bits are a remainder of the node's number: its bits as a polynomial over
// two elements, modulo x^3 + x^2 + 1 (bit i adds kClassOf[i % 7]).  Two nodes next to each other on a lattice, whatever its width
// from 8 to 64, then share a class in 5 % of the cases on average and 11 % at worst (in a diagonal 14 and 24, two columns or rows
// on 5 and 10); with nodes in their own order 6 and 50 (11 and 75, 38 and 77).  Samples left to the candidate pass, 10^6 x 50 on
// 64 x 64 nodes: 254,000 then, 79,000 now (an epoch 1.62 -> 1.41 ms); on 32 x 32 36,000 and 23,000 (422 -> 416 us).  Lattices whose
// own order happens to separate their neighbours lose a little: 20 x 20, 500,000 x 64 1,500 and 6,000 (233 us both), 900,000
// x 25 with distances 300 and 2,500 (154 -> 158 us).  No order that does not know the lattice avoids that: over the widths, a node's
// neighbours in the next row fall into each of eight classes about equally often, so the mean over widths, 0 along the rows and
// 1/8 across, cannot be much below the 6.5 % of this one.
constexpr unsigned class_mask(int bit)                    // the bits of a node's number, from bit 3 on, that flip this bit of its class
{
    constexpr unsigned kClassOf[7] = {1, 2, 4, 5, 7, 3, 6};
    unsigned m = 0u;
    for (int i = 3; i < 32; ++i) m |= ((kClassOf[i % 7] >> bit) & 1u) << i;
    return m;
}
__host__ __device__ __forceinline__ int node_of_row(int row, int K)
{
    if ((row | (kNodesPerStage - 1)) >= K) return row;                       // (a stage with padding rows keeps its order)
    static_assert(kNodesPerStage == 128, "seven bits");
    constexpr unsigned m0 = class_mask(0), m1 = class_mask(1), m2 = class_mask(2);
    const unsigned s = (unsigned)row;
    const unsigned high = (s & ~127u) | (s & 64u) | ((s & 24u) << 1) | ((s & 2u) << 2);      // bits 3 and up of the node
    const unsigned f = (__builtin_popcount(high & m0) & 1) | (__builtin_popcount(high & m1) & 1) << 1 | (__builtin_popcount(high & m2) & 1) << 2;
    return (int)(high | (((s & 1u) | ((s & 4u) >> 1) | ((s & 32u) >> 3)) ^ f));
}

} // namespace som
