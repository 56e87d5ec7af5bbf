// Per-BMU sample sums and counts in LDS with float64 atomics:
//     S_k += x_i,  n_k += 1   for k = b_i       (the inner sums of Eq. 3 grouped by best-matching unit).
//
// Measured on gfx950: ds_add_f64 and the integer LDS atomics complete a 64-lane instruction in about 15 cycles,
// ds_add_f32 needs about 190.  With 8-byte cells the K x (D + 1) partial (the extra column counts samples) does
// not fit one compute unit's LDS, so the NODES are cut into slabs: a workgroup owns a contiguous range of samples
// and one slab of nodes, reads the BMU of every sample of its range (4 bytes), and loads and adds only the rows
// whose BMU falls into its slab.  Every row of X is therefore read exactly once, by exactly one workgroup, as one
// coalesced 64-lane load (lane 0 adds the count, lane l > 0 feature l - 1), followed by one LDS atomic instruction.
// Wavefronts work independently: each reads the BMUs of 256 consecutive samples with one 16-byte load per lane (a
// round ahead), and in four passes of 64 samples takes the rows that belong to the slab off a ballot mask with
// scalar instructions, up to sixteen rows at a time (that many row loads in flight); there is no barrier and no LDS traffic
// other than the atomics inside the range loop.  Where the time goes (10^7 rows of 50 features on 1024 nodes, 431 us
// against 331 us for a kernel that only reads X): a 64-lane LDS atomic takes 15.6 cycles per instruction and COMPUTE
// UNIT whatever its width, 16 cycles a row where the plain read needs 8, and the kernel spends 21; the scan alone
// (every row skipped) costs 64 us for three slabs; more row loads in flight change nothing.  At 10^6 rows, 26 of the
// 57 us do not depend on the rows at all (clearing LDS, the slices, the reduce kernel, two launches).
// At the end the slab moves to the range's slice of a global workspace and a second kernel adds the slices in a
// fixed order.  Counts are exact; the sums are float64 throughout (the order of the atomic additions varies from
// run to run, which moves a sum by a few units in the 16th digit).
// A slab holds every nslabs-th node: nodes that lie together hold similar shares of the samples, and stretches of the nodes' order gave the
// fullest of three slabs 1.2 to 1.6 thirds of them, for which the others' workgroups then waited (10^7 x 50 on a chain of 1024 nodes 586 us and
// 453, 4 * 10^6 listed rows 273 and 253, 10^6 on a lattice, whose few crowded nodes decide, 55 to 60 and 54 to 60 with the reduction).
// The slabs of one sample range get workgroup numbers 8 apart so that they run on the same XCD: rows are not
// aligned to cache lines, and the lines two neighbouring rows share are then fetched into that XCD's L2 once.
#include "som_internal.hpp"

#include <hip/amd_detail/amd_hip_unsafe_atomics.h>

#include <type_traits>

namespace som {

constexpr int kFThreads = 1024;
constexpr size_t kFLdsBytes = 150 * 1024;     // slab

// GATHER: rows are taken through the index list.  A pass's row numbers are one vector load, requested with its ballot, and a row's is
// read off its lane: as a scalar load per row each batch waited for them (10^6 listed rows of 50 features on 1024 nodes 93 -> 80 us).
// R: rows to a load and an LDS instruction.  An LDS atomic takes its 15.6 cycles whatever its width, so rows of up to 15 features
// share one by four and of up to 31 by two: 10^7 x 12 on 1024 nodes 221 -> 193 us, 10^7 x 28 308 -> 286; through a list 439 -> 257
// and 622 -> 412; 10^5 x 5 on 400 17.9 -> 14.5.  (Four rows have eight loads under way: with sixteen their addresses do not fit the
// scalar registers, 10^6 x 8 33 us instead of 30.)
// ONE: one slab, which holds all nodes (dividing node numbers all the same took 3 to 8 % of the kernel: 400,000 x 2 on 4096 nodes 22.2 -> 23.8 us)
template <bool GATHER, int R, bool ONE>
__global__ void __launch_bounds__(kFThreads) accumulate_f64_kernel(const float* __restrict__ X, int D, int64_t ldx,
                                                                   const uint32_t* __restrict__ idx, int64_t m,
                                                                   const int32_t* __restrict__ bmu, int K, int ks,
                                                                   int slabs, int64_t rows_per_range,
                                                                   double* __restrict__ part)
{
    extern __shared__ double f64_lds[];
    const int DS = D + 1, nslabs = ONE ? 1 : slabs;
    double* P = f64_lds;                                                   // [ks][DS]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup number -> (range, slab): slabs of a range sit 8 apart inside a block of 8 * nslabs workgroups
    const int blk = blockIdx.x / (8 * nslabs), within = blockIdx.x % (8 * nslabs);
    const int slab = within / 8;
    const int64_t range = (int64_t)blk * 8 + (within % 8);
    const int kn = ONE ? K : (K - slab + nslabs - 1) / nslabs;                       // nodes of this slab: slab, slab + nslabs, ...
    const int64_t lo = range * rows_per_range;
    if (lo >= m) return;                                   // padding of the last block of 8 ranges (whole workgroup)
    int64_t hi = lo + rows_per_range;
    if (hi > m) hi = m;

    for (int c = tid; c < ks * DS; c += kFThreads) P[c] = 0.0;
    __syncthreads();

    constexpr int G = R == 4 ? 8 : 16;                                           // row loads in flight per wavefront, of R rows each
    constexpr int L = 64 / R;                                             // lanes of a row
    const int fl = lane & (L - 1);
    constexpr int U = 4;                                                  // 64-row passes per load of BMU indices
    // A wavefront takes 64 U consecutive samples at a time: lane l holds the BMUs of samples base + U l .. + U - 1
    // (one 16-byte load, requested a whole round of U passes ahead: with one pass per load the wait for the indices
    // was the longest part of a pass), and pass q works on the samples base + U l + q.
    auto load_bmus = [&](int64_t base, int (&bq)[U]) {
        const int64_t i0 = base + U * lane;
        if (i0 + U <= hi) {
            int4 t;
            __builtin_memcpy(&t, bmu + i0, sizeof(t));
            bq[0] = t.x;
            bq[1] = t.y;
            bq[2] = t.z;
            bq[3] = t.w;
        } else {
#pragma unroll
            for (int q = 0; q < U; ++q) bq[q] = (i0 + q < hi) ? bmu[i0 + q] : -1;
        }
    };
    static_assert(U == 4, "the BMU indices of a round travel as one int4");
    int bq_next[U];
    load_bmus(lo + (int64_t)wave * 64 * U, bq_next);
    const int ldxu = (int)ldx * U;                                         // distance between a pass's rows
    const unsigned recip = 0xffffffffu / (unsigned)nslabs + 1u;            // (exact for node numbers below 2^28: at most sixteen slabs)
    for (int64_t base = lo + (int64_t)wave * 64 * U; base < hi; base += (int64_t)kFThreads * U) {
        int bq[U];
#pragma unroll
        for (int q = 0; q < U; ++q) bq[q] = bq_next[q];
        load_bmus(base + (int64_t)kFThreads * U, bq_next);                 // beyond the range: all -1, nothing is read
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int b = bq[q];
            const unsigned ub = (unsigned)b, at = ONE ? ub : __umulhi(ub, recip);              // b / nslabs
            const bool in = ub < (unsigned)K && (ONE || ub - at * (unsigned)nslabs == (unsigned)slab);
            unsigned long long todo = __ballot(in);                        // wave-uniform: lanes whose row is ours
            const float* xpass = X + (base + q) * ldx;
            const int ncell = (int)at * DS;                                 // this lane's row of P, if its sample is ours
            // Rows are taken off the mask with scalar instructions only (find-first-set, read-lane): no list in
            // LDS, no wait between a row's decoding and its load, so up to G row loads are in flight per wavefront.
            // The scalar unit is shared by the compute unit's wavefronts and this bookkeeping is what it is busy
            // with, so whole batches (sixteen rows, then eight, then four) run without per-row conditions, three
            // scalar instructions a row; what is left of the pass goes through one batch of four places whose empty
            // ones repeat the last row's load and skip the addition.
            int left = __popcll(todo), p_last = 0;
            const int f = fl - 1;                                           // a row's first lane carries the count
            const int fcl = f < 0 ? 0 : (f < D ? f : D - 1);
            const uint32_t row_of_lane = (GATHER && in) ? idx[base + U * lane + q] : 0u;
            // The next R rows of the mask, one to each group of L lanes: the row's first float and its cells.  Behind the last row
            // it is repeated; the group's `live` tells.
            auto take = [&](auto all_there, int& cell, bool& live) -> const float* {
                if constexpr (R == 1) {
                    int p;
                    if constexpr (decltype(all_there)::value) {
                        p = __builtin_ctzll(todo);
                        asm("s_bitset0_b64 %0, %1" : "+s"(todo) : "s"(p));
                        live = true;
                    } else {
                        live = todo != 0ull;
                        p = live ? (int)__ffsll((long long)todo) - 1 : p_last;
                        if (live) {
                            todo &= todo - 1ull;
                            p_last = p;
                        }
                    }
                    cell = __builtin_amdgcn_readlane(ncell, p);
                    // plain variant: 32-bit offset from the pass's first row (63 U rows of ldx floats stay far below 2^31)
                    return GATHER ? X + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)row_of_lane, p) * ldx : xpass + (unsigned)(p * ldxu);
                } else {
                    int c = 0;
                    unsigned at = 0u;
                    live = true;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        int p;
                        bool on = true;
                        if constexpr (decltype(all_there)::value) {
                            p = __builtin_ctzll(todo);
                            asm("s_bitset0_b64 %0, %1" : "+s"(todo) : "s"(p));
                        } else {
                            on = todo != 0ull;
                            p = on ? (int)__ffsll((long long)todo) - 1 : p_last;
                            if (on) {
                                todo &= todo - 1ull;
                                p_last = p;
                            }
                        }
                        const int cp = __builtin_amdgcn_readlane(ncell, p);
                        const unsigned ap = GATHER ? (unsigned)__builtin_amdgcn_readlane((int)row_of_lane, p) : (unsigned)(p * ldxu);
                        const bool mine = lane >= r * L;
                        c = mine ? cp : c;
                        at = mine ? ap : at;
                        live = mine ? on : live;
                    }
                    cell = c;
                    return GATHER ? X + (int64_t)at * ldx : xpass + at;
                }
            };
            auto whole_batch = [&](auto width) {
                constexpr int GB = decltype(width)::value;
                float v[GB];
                int cell[GB];
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    bool live;
                    const float xv = take(std::true_type{}, cell[t], live)[fcl];        // (todo has at least GB R bits set here)
                    v[t] = (fl == 0) ? 1.0f : xv;
                }
                if (fl < DS) {
#pragma unroll
                    for (int t = 0; t < GB; ++t) unsafeAtomicAdd(&P[cell[t] + fl], (double)v[t]);
                }
                left -= GB * R;
            };
            while (left >= G * R) whole_batch(std::integral_constant<int, G>{});
            if (left >= G / 2 * R) whole_batch(std::integral_constant<int, G / 2>{});
            if (left >= G / 4 * R) whole_batch(std::integral_constant<int, G / 4>{});
            if (left > 0) {
                constexpr int GB = G / 4;
                float v[GB];
                int cell[GB];
                bool live[GB];
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    const float xv = take(std::false_type{}, cell[t], live[t])[fcl];
                    v[t] = (fl == 0) ? 1.0f : xv;
                }
#pragma unroll
                for (int t = 0; t < GB; ++t) {
                    if (live[t]) {
                        if (fl < DS) unsafeAtomicAdd(&P[cell[t] + fl], (double)v[t]);
                    }
                }
            }
        }
    }
    __syncthreads();
    // slab -> the range's slice [K][DS], a lane a cell: the slab's rows lie nslabs apart there.  (A row a wavefront left most lanes without a
    // cell on narrow rows: 20,000 x 4 on 4096 nodes 25.8 us, 12.8 this way.)
    double* out = part + (size_t)range * K * DS + (size_t)slab * DS;
    const unsigned recip_row = 0xffffffffu / (unsigned)DS + 1u;            // (exact below 2^26: at most 64 cells a row)
    const int apart = (nslabs - 1) * DS;
    if constexpr (ONE) {
        for (int c = tid; c < K * DS; c += kFThreads) out[c] = P[c];
    } else {
        for (int c = tid; c < kn * DS; c += kFThreads) out[c + (int)__umulhi((unsigned)c, recip_row) * apart] = P[c];
    }
}

// S[k][f] (+)= sum over the ranges' slices, n[k] (+)= sum of their count columns, always in the same order:
// a workgroup takes 64 cells, its four wavefronts a quarter of the slices each, then the quarters are added 0..3.
// D = columns of this launch's feature window, S points at the window's first column, ldS = row length of S; n may
// be null (the counts are taken from the first window only).
__global__ void __launch_bounds__(256) accumulate_f64_reduce_kernel(const double* __restrict__ part, int K, int D,
                                                                    int ranges, int zero_first, double* __restrict__ S,
                                                                    int ldS, unsigned long long* __restrict__ n)
{
    __shared__ double qsum[4][64];
    const int q = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int DS = D + 1;
    const int c = blockIdx.x * 64 + l;
    const int per = (ranges + 3) / 4;
    const int r_lo = q * per, r_hi = (r_lo + per < ranges) ? r_lo + per : ranges;
    double s = 0.0;
    if (c < K * DS) {
        const size_t stride = (size_t)K * DS;
#pragma unroll 8
        for (int r = r_lo; r < r_hi; ++r) s += part[(size_t)r * stride + c];
    }
    qsum[q][l] = s;
    __syncthreads();
    if (q == 0 && c < K * DS) {
        const double tot = ((qsum[0][l] + qsum[1][l]) + qsum[2][l]) + qsum[3][l];
        const int k = c / DS, f = c % DS;
        if (f == 0) {
            if (n) n[k] = (zero_first ? 0ull : n[k]) + (unsigned long long)(tot + 0.5);
        } else {
            S[(size_t)k * ldS + f - 1] = (zero_first ? 0.0 : S[(size_t)k * ldS + f - 1]) + tot;
        }
    }
}

// slabs of LDS that the sums of a map take, one window of features at a time
int accumulate_f64_slabs(int32_t K, int32_t D)
{
    const int ks_max = (int)(kFLdsBytes / ((size_t)((D < 63 ? D : 63) + 1) * sizeof(double)));
    return (K + ks_max - 1) / ks_max;
}

// Returns 1 when the shape is not served by this path (the caller then tries the others), SOM_OK on success, a
// negative code on failure.  Rows wider than 63 features go through in windows of 63 (one kernel + reduce per
// window through the same slices).  Served: a K x 64 float64 partial that fits kFMaxSlabs slabs of LDS.
int accumulate_f64_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m,
                       const int32_t* bmu, int32_t K, double* S, unsigned long long* n, bool zero_first)
{
    if (m <= 0 || ldx >= kFStride) return 1;                // row offsets inside a round of passes are 32-bit
    const int window = D < 63 ? D : 63;                      // features per pass; lane 0 carries the count
    const int nslabs = accumulate_f64_slabs(K, D);
    if (nslabs > kFMaxSlabs) return 1;
    const int ks = (K + nslabs - 1) / nslabs;                  // balanced slabs
    // One workgroup per compute unit and never more workgroups than compute units (with one resident workgroup
    // per unit a grid of 264 ran 60 % slower than one of 240): 256 / nslabs ranges, in whole blocks of 8 so that
    // the slabs of a range share an XCD.
    int64_t ranges = (256 / nslabs) / 8 * 8;
    if (ranges < 8) ranges = 256 / nslabs;
    if (ranges < 1) ranges = 1;
    const int64_t by_rows = (m + kFThreads - 1) / kFThreads;
    if (ranges > by_rows) ranges = by_rows;
    // an odd number of 64-row units per range keeps the range starts off a common power-of-two stride
    int64_t units = ((m + ranges - 1) / ranges + 63) / 64;
    units |= 1;
    const int64_t rows_per_range = units * 64;
    ranges = (m + rows_per_range - 1) / rows_per_range;      // every remaining range holds at least one row
    const int64_t ranges_padded = (ranges + 7) / 8 * 8;
    const size_t need = (size_t)ranges * K * (window + 1) * sizeof(double);
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
    double* part = (double*)ctx->acc_blob;
    const dim3 grid((unsigned)(ranges_padded * nslabs));
    const int together = window < 16 ? 4 : window < 32 ? 2 : 1;          // rows to a load and an addition: as fit 64 lanes
    using Kernel = decltype(&accumulate_f64_kernel<false, 1, false>);
    static constexpr Kernel kernels[2][3][2] = {
#define SOM_F64_KERNELS(R) {accumulate_f64_kernel<false, R, false>, accumulate_f64_kernel<true, R, false>}
#define SOM_F64_KERNELS_ONE(R) {accumulate_f64_kernel<false, R, true>, accumulate_f64_kernel<true, R, true>}
        {SOM_F64_KERNELS(1), SOM_F64_KERNELS(2), SOM_F64_KERNELS(4)}, {SOM_F64_KERNELS_ONE(1), SOM_F64_KERNELS_ONE(2), SOM_F64_KERNELS_ONE(4)}};
#undef SOM_F64_KERNELS
#undef SOM_F64_KERNELS_ONE
    const Kernel kern = kernels[nslabs == 1][together / 2][idx ? 1 : 0];
    if (int rc = check_hip(ctx,
                           hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFLdsBytes),
                           "raising the dynamic LDS limit"))
        return rc;
    for (int f0 = 0; f0 < D; f0 += window) {
        const int dw = (D - f0 < window) ? D - f0 : window;
        const size_t lds = (size_t)ks * (dw + 1) * sizeof(double);
        hipLaunchKernelGGL(kern, grid, dim3(kFThreads), lds, ctx->stream, X + f0, dw, ldx, idx, m, bmu, K, ks, nslabs,
                           rows_per_range, part);
        if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (float64 LDS) launch")) return rc;
        const int cells = K * (dw + 1);
        hipLaunchKernelGGL(accumulate_f64_reduce_kernel, dim3((cells + 63) / 64), dim3(256), 0, ctx->stream, part, K, dw,
                           (int)ranges, zero_first ? 1 : 0, S + f0, D, (f0 == 0) ? n : (unsigned long long*)nullptr);
        if (int rc = check_hip(ctx, hipGetLastError(), "accumulate (float64 LDS) reduce launch")) return rc;
    }
    return SOM_OK;
}

} // namespace som
