// Best-matching-unit search for rows of 65 to 256 features (the default there): a wavefront holds its samples in registers, cut
// into two parts, and the weights, cut the same way, stream through LDS; N x K is never stored.
//
// Arithmetic.  A value is cut into its half-precision part (eleven significant bits) and what that leaves over.  A score takes
// the product of the first parts exactly, on v_mfma_f32_32x32x16_f16, and the two cross products from parts rounded to fp6
// (four bits, one scale for a row), on v_mfma_scale_f32_32x32x64_f8f6f4: its sixty-four places hold [second parts | first parts] of
// thirty-two features on the samples' side and [first parts | second parts] on the weights', so both cross products of a unit of
// 32 features are one MFMA.  Three MFMAs a unit (two and one) where two bf16 parts take six: under the power limit, which bounds both,
// 2 x 21 + 24 ns a unit and SIMD against 6 x 19 (bare loops on random operands).  The error is about 1.9 times that of the
// bf16 parts (2^-12 x 2^-5 four times over, where those drop three terms of 2^-18.5): 5 to 9 % of uniform rows are listed instead
// of 2 to 5.  They are decided by direct float32 differences, so the results are the same.  (The product of the first parts alone
// would list 40 to 80 %.)
//
// Scales.  fp6 has three bits of exponent, half precision five: each sample is scaled by the power of two that takes its largest
// element into [2^11, 2^12), the weights by one that does it for theirs, and the fp6 scales are then constants.  Scores of a sample are
// compared at its scale; what leaves the tile is scaled back.
//
// Tile.  Four wavefronts hold 32 samples each (64 up to 96 features), 14 registers a unit and 32 samples, and walk over the blocks
// of 32 nodes, which are double-buffered in LDS (global_load_lds) with one barrier a block.  Two workgroups share a unit (three at 97 to
// 128 features), so that one brings in its samples (loads, cuts, error norms: 9 to 12 us at 200 features) while the other one's MFMAs
// run.  With 64 samples a wavefront and one workgroup a unit LDS is read half as often, but nothing runs beside that: 10^6 x 200 on
// 1024 nodes 852 us, 766 this way (1015 with the compiler's copies between the halves of the register file, 1600 by the 256 x 256
// tiles of som_bmu_wide.hip, which cut every sample once for each 256 nodes).
// What bounds it: the power limit (at 4096 nodes the clock is at 1.55 to 1.7 GHz with the matrix pipes busy 0.55 to 0.59 of the time; at 1024 1.6 GHz
// and 0.48), and waits: at 1024 nodes neither pipe works in a third of the cycles.  Without the fold the loop takes 9 % less, without its LDS reads 2 %.
#include "som_bmu_common.hpp"
#include "som_bmu_wide.hpp"

#include <math.h>

namespace som {

constexpr int kHThreads = 256;
constexpr int kHWaves = kHThreads / 64;
constexpr int kHAhead = 3;                         // groups of MFMAs between a fragment's read from LDS and its use
constexpr int kHRange = 30;                        // largest difference of the samples' and the weights' scales
constexpr float kHPadNorm = -1.2379400e+27f;       // -2^90: padding rows; times 2^-30 .. 2^30 still below any score

constexpr int held_ms(int H) { return H > 3 ? 1 : 2; }        // blocks of 32 samples of a wavefront
constexpr int held_waves(int H) { return H == 4 ? 3 : 2; }    // workgroups on a unit (registers)
constexpr int held_tile_rows(int H) { return kHWaves * 32 * held_ms(H); }
constexpr int held_units(int D) { return (D + 31) / 32; }
constexpr int held_block_bytes(int H) { return (H * 3584 + 1023) / 1024 * 1024; }

// 64 lanes x 4 bytes, as lds_load16
__device__ __forceinline__ void lds_load4(const void* from, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(from) : "memory", "m0");
}

// ---------------------------------------------------------------------------------------------------------
// Weight preparation: a wavefront a row of the blocks (node_of_row: neighbours on the map into different classes) cuts it and
// sums what the cuts leave over; the rest of the grid writes the transposed copy that the all-nodes pass reads.
// ---------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) bmu_held_prep_kernel(const float* __restrict__ W, int K, int D, int kpad, int H,
                                                            const float* __restrict__ centre, const float* __restrict__ spread,
                                                            char* __restrict__ blob, float* __restrict__ hats, float* __restrict__ norms,
                                                            float* __restrict__ wt, unsigned int* __restrict__ scal,
                                                            double* __restrict__ qe, int32_t* __restrict__ small)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < 2 && qe) qe[e] = 0.0;
    if (e < 4 && small) small[e] = 0;
    const int node_groups = kpad / 4;                          // workgroups that take four rows each
    if ((int)blockIdx.x >= node_groups) {
        const int64_t t = (int64_t)(blockIdx.x - node_groups) * 256 + threadIdx.x;
        if (t < (int64_t)D * kpad) {
            const int f = (int)(t / kpad), k = (int)(t - (int64_t)f * kpad);
            wt[t] = k < K ? W[(size_t)k * D + f] : 0.0f;
        }
        return;
    }
    __shared__ __align__(16) _Float16 part[4][2][kHeldFeatures];
    __shared__ float most[4][4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 4 + wave, k = node_of_row(r, K);
    // place `slot` of a row: features in fours, the last ones shifted back into the row (own features only, zeros in front of them)
    float w[kHeldFeatures / 64], c[kHeldFeatures / 64];
#pragma unroll
    for (int i = 0; i < kHeldFeatures / 64; ++i) {
        const int slot = lane + 64 * i, q = slot >> 2, start = 4 * q < D - 4 ? 4 * q : D - 4, f = start + (slot & 3);
        const bool own = k < K && f >= 4 * q;
        w[i] = own ? W[(size_t)k * D + f] : 0.0f;
        c[i] = own ? centre[f] : 0.0f;
    }
    float top = 0.0f;
#pragma unroll
    for (int b = 0; b < kHeldFeatures / 64; ++b) top = fmaxf(top, 64 * b < D ? spread[b] : 0.0f);
    const int sw = scale_for(top);
    if (e == 0) scal[kScalShift] = (unsigned)sw;
    const float s = power_of_two(sw);
    double nrm = 0.0;
    float lo2 = 0.0f, over = 0.0f;
#pragma unroll
    for (int i = 0; i < kHeldFeatures / 64; ++i) {
        const int slot = lane + 64 * i;
        if (slot < 32 * H) {
            const float v = w[i] - c[i];
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
    }
    nrm = wave_sum(nrm);
    __syncthreads();
    const int R = r & 31;
    char* const to = blob + (size_t)(r >> 5) * held_block_bytes(H);
    if (lane < 4 * H) {
        const int u = lane >> 2, kb = (lane >> 1) & 1, g = lane & 1;
        *reinterpret_cast<uint4*>(to + u * 3072 + kb * 1024 + (g * 32 + R) * 16) =
            *reinterpret_cast<const uint4*>(&part[wave][0][32 * u + 16 * kb + 8 * g]);
    }
    float q2 = 0.0f;
    if (lane < 2 * H) {
        const int u = lane >> 1, g = lane & 1;               // the first lane half feeds first parts, the other one second parts
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
        *reinterpret_cast<uint4*>(to + u * 3072 + 2048 + (g * 32 + R) * 16) = make_uint4(q[0], q[1], q[2], q[3]);
        *reinterpret_cast<uint2*>(to + H * 3072 + u * 512 + (g * 32 + R) * 8) = make_uint2(q[4], q[5]);
    }
    float qh2 = (lane & 1) == 0 ? q2 : 0.0f, ql2 = (lane & 1) == 1 ? q2 : 0.0f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo2 += __shfl_xor(lo2, o);
        over += __shfl_xor(over, o);
        qh2 += __shfl_xor(qh2, o);
        ql2 += __shfl_xor(ql2, o);
    }
    if (lane == 0) {
        const float back = power_of_two(-sw);
        const double full = -0.5 * nrm * (double)s * (double)s;
        hats[r] = k < K && full > (double)kHPadNorm ? (float)full : kHPadNorm;
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

// H: units of 32 features; SHORT: the last one has sixteen at most, so that its other sixteen need no MFMA of first parts (10^6 x 200 on 1024
// nodes, one of 21: 853 -> 842 us; zeros draw little power, and the clock is at the power limit)
template <int H, bool SHORT>
struct HeldArgs {
    // [block of 32 rows][unit][first parts of 16 features | of the other 16 | fp6, 16 of a lane's 24 bytes], then [unit][fp6, the other 8]: in the
    // order of the lanes, rounded up to whole kilobytes
    const char* blob;
    const float* hats;       // [kpad] -|w|^2 / 2 at the weights' scale, in the order of the rows
    int blocks;              // blocks of 32 rows that hold a node
};

// Blocks [b_lo, b_hi) (b_lo even) for the samples of tile `tile`.  CAND: the samples are the entries of the re-decision list, and every
// node that reaches the entry's cut is appended to its record; the scores are those of the search bit for bit.
template <int H, bool SHORT, bool CAND>
__device__ __forceinline__ void held_tile(const BmuArgs& a, const WideArgs& p, const HeldArgs<H, SHORT>& hp, int64_t tile, int split, int b_lo, int b_hi,
                                          int64_t total, char* lds)
{
    constexpr int MS = held_ms(H);
    constexpr int GROUPS = 3 * H;
    constexpr int BLK = held_block_bytes(H);
    constexpr int AHEAD = kHAhead;
    static_assert(GROUPS % AHEAD == 0, "a fragment's place is its group's number modulo the distance");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 31, g = lane >> 5;
    const int64_t wave0 = (tile * kHWaves + wave) * (32 * MS);
    // LDS: [2][BLK] blocks, [4][64] norms of blocks, [32 H] centre
    float* const ring = reinterpret_cast<float*>(lds + 2 * BLK);
    float* const centre = ring + 4 * 64;
    const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char*)lds);

    auto load_block = [&](int b) {
        const char* from = hp.blob + (size_t)b * BLK + lane * 16;
        const unsigned to = lds0 + (unsigned)(b & 1) * BLK;
#pragma unroll
        for (int i = 0; i < (BLK / 1024 + kHWaves - 1) / kHWaves; ++i) {
            const int q = wave + kHWaves * i;
            if (q < BLK / 1024) lds_load16(from + q * 1024, to + q * 1024);
        }
        // (lanes behind the thirty-second read the block's norms a second time, which nobody looks at)
        if (wave == kHWaves - 1) lds_load4(hp.hats + b * 32 + j, lds0 + 2 * BLK + (unsigned)(b & 3) * 256);
    };
    load_block(b_lo);
    if (tid < 32 * H) centre[tid] = tid < a.D ? a.centre[tid] : 0.0f;
    static_assert(32 * H <= kHThreads, "an entry a thread");
    if (tid < 64) ring[((b_lo - 1) & 3) * 64 + tid] = 0.0f;          // (the norms of the set that the first block folds)

    // ---- this wavefront's samples
    const int sw = (int)a.scal[kScalShift];
    const float* row[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
        int64_t i = wave0 + mb * 32 + j;
        i = i < total ? i : total - 1;
        if constexpr (CAND) i = (int64_t)a.recheck[i];
        row[mb] = a.X + (a.idx ? (int64_t)a.idx[i] : i) * a.ldx;
    }
    auto start_of = [&](int u, int kb, int h) {
        const int f0 = 32 * u + 16 * kb + 8 * g + 4 * h;
        return u < H - 1 ? f0 : f0 < a.D - 4 ? f0 : a.D - 4;
    };
    float v[MS][H][2][8];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb)
#pragma unroll
        for (int u = 0; u < H; ++u)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const float4 t = SHORT && u == H - 1 && kb == 1 ? make_float4(0.f, 0.f, 0.f, 0.f) : load4(row[mb] + start_of(u, kb, h));
                    v[mb][u][kb][4 * h + 0] = t.x;
                    v[mb][u][kb][4 * h + 1] = t.y;
                    v[mb][u][kb][4 * h + 2] = t.z;
                    v[mb][u][kb][4 * h + 3] = t.w;
                }
    __syncthreads();                               // (the centre)
    halfx8 xf[MS][H][2];
    uintx6 xq[MS][H];
    float fx[MS];             // 2^(scale of the sample - scale of the weights)
    float back[MS];           // 2^-(scale of the sample)
    float cut[MS];
    int64_t entry[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
        int64_t i = wave0 + mb * 32 + j;
        const bool real = i < total;
        i = real ? i : total - 1;
        if constexpr (CAND) {
            cut[mb] = real ? a.cutv[i] : NAN;               // no score compares >= NaN
            i = (int64_t)a.recheck[i];
        }
        entry[mb] = i;
        float most = 0.0f;
#pragma unroll
        for (int u = 0; u < H; ++u)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (SHORT && u == H - 1 && kb == 1) continue;
                    const int start = start_of(u, kb, h);
                    const float4 c = load4(centre + start);
                    const float cc[4] = {c.x, c.y, c.z, c.w};
                    // (windows shifted back at the end of the row: own elements only)
                    const int shift = 32 * u + 16 * kb + 8 * g + 4 * h - start;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        float& x = v[mb][u][kb][4 * h + t];
                        x -= cc[t];
                        if (u == H - 1) x = shift <= t ? x : 0.0f;
                    }
                    most = fmaxf(most, fmaxf(fmaxf(fabsf(v[mb][u][kb][4 * h]), fabsf(v[mb][u][kb][4 * h + 1])),
                                             fmaxf(fabsf(v[mb][u][kb][4 * h + 2]), fabsf(v[mb][u][kb][4 * h + 3]))));
                }
        most = fmaxf(most, __shfl_xor(most, 32));
        int sx = scale_for(most);
        sx = sx < sw - kHRange ? sw - kHRange : sx > sw + kHRange ? sw + kHRange : sx;
        const float s = power_of_two(sx);
        fx[mb] = power_of_two(sx - sw);
        const float back_x = power_of_two(-sx);
        back[mb] = back_x;
        if constexpr (CAND) cut[mb] = cut[mb] * s * power_of_two(sw);
        const float q_scale = g == 0 ? power_of_two(-3) : power_of_two(kTopBit - 2);
        float v2 = 0.0f, e2 = 0.0f, after2 = 0.0f;
#pragma unroll
        for (int u = 0; u < H; ++u) {
            unsigned int hi[8], lo[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float x0 = v[mb][u][t >> 2][2 * (t & 3)] * s, x1 = v[mb][u][t >> 2][2 * (t & 3) + 1] * s;
                const HalfPair h(x0, x1);
                hi[t] = h.hi;
                lo[t] = h.lo;
            }
            xf[mb][u][0] = __builtin_bit_cast(halfx8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            xf[mb][u][1] = __builtin_bit_cast(halfx8, make_uint4(hi[4], hi[5], hi[6], hi[7]));
            // the first lane half packs the second parts of all thirty-two features, the other half the first parts
            uintx16 w;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                unsigned int m = lo[t], n = hi[t];
                swap_words(m, n);
                w[t] = m;
                w[8 + t] = n;
            }
            const halfx32 own = __builtin_bit_cast(halfx32, w);
            const uintx6 q = __builtin_amdgcn_cvt_scalef32_pk32_fp6_f16(own, q_scale);
            xq[mb][u] = q;
            if constexpr (!CAND) {
                const uintx16 d = __builtin_bit_cast(uintx16, __builtin_amdgcn_cvt_scalef32_pk32_f16_fp6(q, q_scale));
                float s2 = 0.0f;
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    const halfx2 o = __builtin_bit_cast(halfx2, (unsigned int)w[t]);
                    const halfx2 r = o - __builtin_bit_cast(halfx2, (unsigned int)d[t]);
                    s2 = __builtin_amdgcn_fdot2(o, o, s2, false);
                    e2 = __builtin_amdgcn_fdot2(r, r, e2, false);
                }
                v2 += s2;
                const float after = (float)(2 * (H - u));        // MFMAs from its own on
                after2 = fmaf(after * after, s2, after2);
            }
        }
        if constexpr (!CAND) {
            // the lower half of the lanes has the second parts' sums, the upper half the first parts'
            const float h2 = __shfl_xor(v2, 32), eh2 = __shfl_xor(e2, 32), ha2 = __shfl_xor(after2, 32);
            if (split == 0 && g == 0 && real) p.norm[i] = part_norms(a, v2, e2, h2, eh2, ha2, (float)(H + 2), 0.0f, back_x, power_of_two(-sw));
        }
    }

    constexpr int CLS = CAND ? 1 : 4;
    float best[MS][CLS], second[MS][CLS];
    int from[MS][CLS];
    unsigned int found[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb) {
        found[mb] = 0u;
#pragma unroll
        for (int c = 0; c < CLS; ++c) {
            best[mb][c] = -INFINITY;
            second[mb][c] = -INFINITY;
            from[mb][c] = 0;
        }
    }
    // One fold step takes scores r and r + 2 of sample block mb, in three parts of three vector instructions, so that every MFMA
    // has its share behind it.
    // (quads of rows, the samples' blocks in turn: a quad's norms wait in four registers)
    float before[MS][2], t0, t1;
    float4 nrm[2];
    const float4* n4 = nullptr;
    auto fold_part = [&](const floatx16 (&s)[MS], int at, auto par, int b) {
        const int step = at / 3, part = at % 3;
        const int quad = step / (2 * MS), mb = (step >> 1) % MS, c = step & 1, r0 = 4 * quad + c, r1 = r0 + 2;
        const float4& n = nrm[quad & 1];
        if (part == 0) {
            t0 = fmaf(c ? n.y : n.x, fx[mb], s[mb][r0]);
            t1 = fmaf(c ? n.w : n.z, fx[mb], s[mb][r1]);
            if (step % (2 * MS) == 2 * MS - 1 && quad < 2) nrm[quad & 1] = n4[2 * (quad + 2)];
            if constexpr (!CAND) t0 = __uint_as_float((__float_as_uint(t0) & 0xfffffff8u) | (unsigned)(r0 >> 1));
        } else if constexpr (CAND) {
            if (part == 1) {
                found[mb] = 2u * found[mb] + (t0 >= cut[mb] ? 1u : 0u);
                found[mb] = 2u * found[mb] + (t1 >= cut[mb] ? 1u : 0u);
            } else if (r1 == 15) {
                if (found[mb] != 0u) {
                    uint32_t* rec = p.record + entry[mb] * kWRecord;
                    for (unsigned int bits = found[mb]; bits != 0u;) {
                        const int bit = 31 - __builtin_clz(bits), place = 15 - bit;
                        bits ^= 1u << bit;
                        const int r = 4 * (place >> 2) + ((place >> 1) & 1) + 2 * (place & 1);
                        const int id = node_of_row(b * 32 + 8 * (r >> 2) + 4 * g + (r & 3), a.K);
                        const unsigned at = atomicAdd(rec, 1u);
                        if (at < (unsigned)kWIds) reinterpret_cast<uint16_t*>(rec + 1)[at] = (uint16_t)id;
                    }
                    found[mb] = 0u;
                }
            }
        } else {
            const int k = 2 * decltype(par)::value + c;
            if (part == 1) {
                if (r0 < 2) before[mb][c] = best[mb][k];
                t1 = __uint_as_float((__float_as_uint(t1) & 0xfffffff8u) | (unsigned)(r1 >> 1));
                const float mid = __builtin_amdgcn_fmed3f(best[mb][k], t0, t1);
                second[mb][k] = vmax(second[mb][k], mid);
            } else {
                best[mb][k] = vmax3(best[mb][k], t0, t1);
                if (r1 >= 14) from[mb][k] = best[mb][k] > before[mb][c] ? b : from[mb][k];
            }
        }
    };

    // ---- fragments of the weights: group i is unit i's small products, then first parts, two MFMAs a unit
    uintx6 fa[AHEAD];
    const int lane16 = lane * 16, lane8 = H * 3072 + lane * 8;
    auto read = [&](const char* base, int i) {
        uintx6& f = fa[i % AHEAD];
        const uint4 t = *reinterpret_cast<const uint4*>(base + lane16 + (i < H ? i * 3072 + 2048 : ((i - H) >> 1) * 3072 + ((i - H) & 1) * 1024));
        f[0] = t.x;
        f[1] = t.y;
        f[2] = t.z;
        f[3] = t.w;
        if (i < H) {
            const uint2 r = *reinterpret_cast<const uint2*>(base + lane8 + i * 512);
            f[4] = r.x;
            f[5] = r.y;
        }
    };
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    const int scale_a = g == 0 ? 127 + kTopBit - 2 : 127 - 3, scale_b = g == 0 ? 127 - 3 : 127 + kTopBit - 2;
    constexpr int USED = SHORT ? GROUPS - 1 : GROUPS;          // (the last group's place in the schedule stays)
    constexpr int PARTS = 3 * 8 * MS, MFMAS = USED * MS;
    auto block = [&](floatx16 (&cur)[MS], const floatx16 (&prev)[MS], auto prev_par, int b) {
        const char* base = lds + (b & 1) * BLK;
        const char* next = lds + ((b + 1) & 1) * BLK;
        n4 = reinterpret_cast<const float4*>(ring + ((b - 1) & 3) * 64) + g;
        nrm[0] = n4[0];
        nrm[1] = n4[2];
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) {
            const bool small_products = i < H;
            const int u = small_products ? i : (i - H) >> 1, kb = (i - H) & 1;
#pragma unroll
            for (int mb = 0; mb < MS; ++mb) {
                if (i >= USED) continue;
                if (small_products) {
                    cur[mb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fp6_operand(fa[i % AHEAD]), fp6_operand(xq[mb][u]), i == 0 ? zero16 : cur[mb], 2,
                                                                              2, 0, scale_a, 0, scale_b);
                } else {
                    const uintx4 w = __builtin_shufflevector(fa[i % AHEAD], fa[i % AHEAD], 0, 1, 2, 3);
                    cur[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, w), xf[mb][u][kb], cur[mb], 0, 0, 0);
                }
                const int m = i * MS + mb;
#pragma unroll
                for (int f = m * PARTS / MFMAS; f < (m + 1) * PARTS / MFMAS; ++f) fold_part(prev, f, prev_par, b - 1);
                if (mb + 1 < MS) __builtin_amdgcn_sched_barrier(0);
            }
            if (i + AHEAD < GROUPS) {
                if (i + AHEAD < USED) read(base, i + AHEAD);
            } else if (i + AHEAD == GROUPS) {
                // Everything of this block has been read: its place goes to the block after next, and the next one, on its way
                // since a block ago, has to be there.
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if (b + 2 < b_hi) load_block(b + 2);
                read(next, 0);
            } else {
                read(next, i + AHEAD - GROUPS);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (b_lo + 1 < b_hi) load_block(b_lo + 1);
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) read(lds + (b_lo & 1) * BLK, i);
    floatx16 accA[MS], accB[MS];
#pragma unroll
    for (int mb = 0; mb < MS; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) accB[mb][r] = kSplitPadNorm;          // (the first block folds a set that no real score is below)
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    int b = b_lo;                                  // (even)
    for (; b + 1 < b_hi; b += 2) {
        block(accA, accB, Odd{}, b);
        block(accB, accA, Even{}, b + 1);
    }
    const bool odd = b < b_hi;
    if (odd) block(accA, accB, Odd{}, b);
    {
        const int last = b_hi - 1;
        n4 = reinterpret_cast<const float4*>(ring + (last & 3) * 64) + g;
        nrm[0] = n4[0];
        nrm[1] = n4[2];
        if (odd) {
#pragma unroll
            for (int f = 0; f < PARTS; ++f) fold_part(accA, f, Even{}, last);
        } else {
#pragma unroll
            for (int f = 0; f < PARTS; ++f) fold_part(accB, f, Odd{}, last);
        }
    }
    if constexpr (CAND) return;

    // ---- lane (j, g) finishes sample j of block g: the halves trade what they hold of each other's block
    auto swap_f = [](float& x, float& y) {
        unsigned int m = __float_as_uint(x), n = __float_as_uint(y);
        swap_words(m, n);
        x = __uint_as_float(m);
        y = __uint_as_float(n);
    };
    float won[8];
    int where[8];
#pragma unroll
    for (int c = 0; c < CLS; ++c) {
        won[c] = best[0][c];
        won[4 + c] = best[MS - 1][c];
        swap_f(won[c], won[4 + c]);
        unsigned int m = (unsigned)from[0][c], n = (unsigned)from[MS - 1][c];
        swap_words(m, n);
        where[c] = (int)m;
        where[4 + c] = (int)n;
    }
    float m0 = fmaxf(fmaxf(second[0][0], second[0][1 % CLS]), fmaxf(second[0][2 % CLS], second[0][3 % CLS]));
    float m1 = fmaxf(fmaxf(second[MS - 1][0], second[MS - 1][1 % CLS]), fmaxf(second[MS - 1][2 % CLS], second[MS - 1][3 % CLS]));
    swap_f(m0, m1);
    const int64_t i = wave0 + (MS > 1 ? lane : j);
    const float un = g == 0 ? back[0] : back[MS - 1], uw = power_of_two(-sw);      // (this lane's sample is of block g)
    if (i < total && (MS > 1 || g == 0)) write_winners(a, p, split, i, won, where, fmaxf(m0, m1), un * uw);
}

template <int H, bool SHORT>
__device__ __forceinline__ void held_search(const BmuArgs& a, const WideArgs& p, const HeldArgs<H, SHORT>& hp, char* lds)
{
    const int64_t blk = blockIdx.x / (8 * p.splits);
    const int within = (int)(blockIdx.x % (8 * p.splits));
    const int64_t tile = blk * 8 + within % 8;
    const int split = within / 8;
    if (tile * held_tile_rows(H) >= a.m) return;
    const int b_lo = split * p.per_split, b_hi = b_lo + p.per_split < hp.blocks ? b_lo + p.per_split : hp.blocks;
    held_tile<H, SHORT, false>(a, p, hp, tile, split, b_lo, b_hi, a.m, lds);
}

// A fixed grid walks the (tile of the list, range of blocks) units: as many ranges as keep it busy.
template <int H, bool SHORT>
__device__ __forceinline__ void held_candidates(const BmuArgs& a, const WideArgs& p, const HeldArgs<H, SHORT>& hp, char* lds)
{
    const unsigned int count = a.scal[a.slot];
    if (count <= p.cand_min) return;
    const int tiles = (int)((count + held_tile_rows(H) - 1) / held_tile_rows(H));
    int ranges = ((int)gridDim.x + tiles - 1) / tiles;
    const int pairs = (hp.blocks + 1) / 2;
    int per = 2 * ((pairs + ranges - 1) / ranges);
    per = per < 8 ? 8 : per;
    ranges = (hp.blocks + per - 1) / per;
    for (int64_t u = blockIdx.x; u < (int64_t)tiles * ranges; u += gridDim.x) {
        const int b_lo = (int)(u % ranges) * per, b_hi = b_lo + per < hp.blocks ? b_lo + per : hp.blocks;
        held_tile<H, SHORT, true>(a, p, hp, u / ranges, 0, b_lo, b_hi, (int64_t)count, lds);
        __syncthreads();
    }
}

// (overloads of the wide search's two kernels, one for each number of units and kind of the last)
#define SOM_HELD_KERNELS(H, SHORT)                                                                                                                 \
    __global__ void __launch_bounds__(kHThreads) __attribute__((amdgpu_waves_per_eu(held_waves(H), held_waves(H))))                                \
    bmu_wide_split_kernel(const BmuArgs a, const WideArgs p, const HeldArgs<H, SHORT> hp)                                                          \
    {                                                                                                                                              \
        extern __shared__ float4 held_lds[];                                                                                                       \
        held_search(a, p, hp, reinterpret_cast<char*>(held_lds));                                                                                  \
    }                                                                                                                                              \
    __global__ void __launch_bounds__(kHThreads) __attribute__((amdgpu_waves_per_eu(held_waves(H), held_waves(H))))                                \
    bmu_wide_split_cand_kernel(const BmuArgs a, const WideArgs p, const HeldArgs<H, SHORT> hp)                                                     \
    {                                                                                                                                              \
        extern __shared__ float4 held_lds[];                                                                                                       \
        held_candidates(a, p, hp, reinterpret_cast<char*>(held_lds));                                                                              \
    }
#define SOM_HELD_BOTH(H) SOM_HELD_KERNELS(H, false) SOM_HELD_KERNELS(H, true)
SOM_HELD_BOTH(3)
SOM_HELD_BOTH(4)
SOM_HELD_BOTH(5)
SOM_HELD_BOTH(6)
SOM_HELD_BOTH(7)
SOM_HELD_BOTH(8)
#undef SOM_HELD_BOTH
#undef SOM_HELD_KERNELS

// ---------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------
static size_t held_blob(int32_t kpad, int32_t D) { return (size_t)(kpad / 32) * held_block_bytes(held_units(D)); }

size_t bmu_held_blob_bytes(int32_t kpad, int32_t D)
{
    return held_blob(kpad, D) + (2 * (size_t)kpad + 64) * sizeof(float);
}

float* bmu_held_spread(const BmuPrep& prep, int32_t D)
{
    return (float*)((char*)prep.stage16 + held_blob(prep.kpad, D)) + 2 * (size_t)prep.kpad;
}

int bmu_held_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small)
{
    char* blob = (char*)prep.stage16;
    float* hats = (float*)(blob + held_blob(prep.kpad, D));
    const int64_t groups = prep.kpad / 4 + ((int64_t)D * prep.kpad + 255) / 256;
    hipLaunchKernelGGL(bmu_held_prep_kernel, dim3((unsigned)groups), dim3(256), 0, ctx->stream, W, K, D, prep.kpad, held_units(D), prep.centre,
                       bmu_held_spread(prep, D), blob, hats, hats + prep.kpad, prep.wt, prep.scal, qe, small);
    return check_hip(ctx, hipGetLastError(), "bmu (held rows) preparation launch");
}

// Workgroups per sample tile, as for the tile (som_bmu_wide.hip): bringing in a tile's samples takes as long as about ten blocks.  (The last,
// partial round split further, as in som_bmu_cut.hip, gives nothing here: 10^5 x 80, 120 and 200 on 1024 nodes 361 us for 360, 509 for 501,
// 798 for 792.)
void bmu_held_plan(WideArgs& p, const BmuPrep& prep, int64_t m, int32_t K, int32_t D, int units)
{
    const int H = held_units(D), rows = held_tile_rows(H), blocks = (K + 31) / 32;
    const int64_t tiles = (m + rows - 1) / rows;
    p.norms = (const float*)((const char*)prep.stage16 + held_blob(prep.kpad, D)) + prep.kpad;
    units *= held_waves(H);
    int best = 1, steps = (blocks + 1) / 2 * 2;
    double best_cost = 0.0;
    for (int s = 1; s <= 16 && 2 * s <= blocks + 1; ++s) {
        const int per = ((blocks + s - 1) / s + 1) / 2 * 2;
        if ((blocks + per - 1) / per != s) continue;
        const double cost = (double)((tiles * s + units - 1) / units) * ((double)per + 10.0);
        if (s == 1 || cost < best_cost * 0.98) {
            best = s;
            steps = per;
            best_cost = cost;
        }
    }
    p.set_splits(m, best, steps, (tiles + 7) / 8 * 8 * best);
}

template <int H, bool SHORT>
static HeldArgs<H, SHORT> held_args(const BmuPrep& prep, const BmuArgs& a)
{
    HeldArgs<H, SHORT> h{};
    h.blob = (const char*)prep.stage16;
    h.hats = (const float*)(h.blob + held_blob(prep.kpad, a.D));
    h.blocks = (a.K + 31) / 32;
    return h;
}

template <int H, bool SHORT>
static int launch_held(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, const WideArgs& p, bool cand)
{
    constexpr size_t lds = 2 * (size_t)held_block_bytes(H) + (4 * 64 + 32 * H) * sizeof(float);
    static_assert(lds <= 65536, "offsets of global_load_lds below 64 KB");
    const HeldArgs<H, SHORT> h = held_args<H, SHORT>(prep, a);
    using Kernel = void (*)(const BmuArgs, const WideArgs, const HeldArgs<H, SHORT>);
    const Kernel search = bmu_wide_split_kernel, candidates = bmu_wide_split_cand_kernel;
    if (cand)
        hipLaunchKernelGGL(candidates, dim3(256 * held_waves(H)), dim3(kHThreads), lds, ctx->stream, a, p, h);
    else
        hipLaunchKernelGGL(search, dim3((unsigned)p.grid), dim3(kHThreads), lds, ctx->stream, a, p, h);
    return check_hip(ctx, hipGetLastError(), "bmu (held rows) launch");
}

int bmu_held_launch(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, const WideArgs& p, bool cand)
{
    const int last = (a.D - 1) % 32 + 1;                       // features of the last unit
    switch (2 * held_units(a.D) + (last <= 16 ? 1 : 0)) {
    case 6: return launch_held<3, false>(ctx, prep, a, p, cand);
    case 7: return launch_held<3, true>(ctx, prep, a, p, cand);
    case 8: return launch_held<4, false>(ctx, prep, a, p, cand);
    case 9: return launch_held<4, true>(ctx, prep, a, p, cand);
    case 10: return launch_held<5, false>(ctx, prep, a, p, cand);
    case 11: return launch_held<5, true>(ctx, prep, a, p, cand);
    case 12: return launch_held<6, false>(ctx, prep, a, p, cand);
    case 13: return launch_held<6, true>(ctx, prep, a, p, cand);
    case 14: return launch_held<7, false>(ctx, prep, a, p, cand);
    case 15: return launch_held<7, true>(ctx, prep, a, p, cand);
    case 16: return launch_held<8, false>(ctx, prep, a, p, cand);
    case 17: return launch_held<8, true>(ctx, prep, a, p, cand);
    }
    return fail(ctx, SOM_EINVAL, "no kernel for held rows of %d features", a.D);
}

} // namespace som
