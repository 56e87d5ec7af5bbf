// Best-matching-unit search for rows of more than 256 features on small maps, and what it shares with the other two searches of rows wider
// than 64 (bmu_wide_form): the join, the direct differences and the host side.  The scores are those of bmu_split_kernel
// (som_bmu.hip: samples and weights cut into two bf16 parts, three bf16 MFMA products per float32 product) as a tiled
// matrix product with the running arg-max behind it; N x K is never stored.
//
// Tile.  A workgroup of eight wavefronts forms 256 samples x 256 nodes at a time, features in chunks of 32; a wavefront
// owns 64 samples x 128 nodes (four node blocks of 32, taken alternately by the two wavefronts of the same samples).
// Per chunk it reads 12 + 4 fragments from LDS per 24 MFMAs, which keeps LDS at about half its rate; tiles of one block
// of 32 samples per wavefront, as in the kernel before this one, read their samples' parts from memory once per 128
// nodes, 32 bytes a lane at a stride of a whole row, and ran at a quarter of the matrix rate.
//
// Data path.  The weights are cut once per preparation and stored in the order in which the MFMA's lanes take them, so a
// chunk of a node tile is 32 KB that go straight from memory to LDS (global_load_lds_dwordx4).  The samples are read in
// float32, 128 contiguous bytes of a row per four lanes, centred, cut and written to LDS by the workgroup itself, for
// every node tile again, beside the MFMAs; a conversion pass of its own moves every row twice more through memory (386 us at
// 10^6 x 200; the tile, with both operands straight from memory, then took 1410 us instead of 1581: dropped).  Both operands are
// double-buffered; one barrier per chunk.  Chunks run on without a break across node tiles: a tile's scores are folded
// while the next tile's first chunk is on the matrix pipe.
// What bounds it is neither pipe alone: at 10^6 x 200 on 1024 nodes the matrix pipes are busy 42 % of the time and the vector units, with 6.9
// instructions for each MFMA (of a wavefront's 331 a chunk, 128 add the chunk's products up), 36 %, but only a quarter of those run
// beside an MFMA, and for 30 % of the time neither works; an MFMA takes 36 to 39 ns where the probe sustains 23 with six vector
// instructions beside each, and the clock stays at 2.24 GHz.
//
// Accumulation.  A chunk's products are summed on their own from zero, the small ones (lo hi, hi lo) first, and then
// added to the tile's accumulators: the roundings inside a chunk are relative to |x_chunk| |w_chunk|, which add up to at
// most |x| |w| over the chunks (Cauchy-Schwarz), instead of growing with the number of features.
//
// After the tiles, bmu_wide_join_kernel takes every sample's winners over the node tiles, its error bound from the norms
// formed on the way, and decides which samples are open: those whose candidates are all known get their ids written
// down, the others go through the tile kernel again (CAND), which notes every node that reaches the sample's cut.
// bmu_wide_exact_kernel decides both by direct float32 differences, and what it cannot serve is left to the all-nodes pass.
#include "som_bmu_wide.hpp"

#include <math.h>

#include <type_traits>

namespace som {

// Eight values as two bf16 parts each, one by one.  (As pairs, which is what the narrow search's prologue takes, this tile has eleven
// registers spilled instead of five, and 10^6 x 200 on 1024 nodes takes 1 to 2 % longer.)
__device__ __forceinline__ void cut8(const float (&v)[8], bf16x8& hi, bf16x8& lo)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        hi[i] = (__bf16)v[i];
        lo[i] = (__bf16)(v[i] - (float)hi[i]);
    }
}
// the same, and what the first parts leave over is added to left2 (squares)
__device__ __forceinline__ void cut8(const float (&v)[8], bf16x8& hi, bf16x8& lo, float& left2)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        hi[i] = (__bf16)v[i];
        const float left = v[i] - (float)hi[i];
        lo[i] = (__bf16)left;
        left2 = fmaf(left, left, left2);
    }
}

constexpr int kWThreads = 512;
constexpr int kWTile = 256;                       // samples, and nodes, of a tile
constexpr int kWChunk = 32;                       // features of a chunk
constexpr int kWBuf = kWTile * kWChunk * 4;       // bytes of an operand's chunk in LDS (hi and lo parts)
constexpr int kWState = 12;                       // words of running state per lane
constexpr size_t kWLds = 4 * (size_t)kWBuf + (kWThreads * kWState + kWTile) * sizeof(float);
// ---------------------------------------------------------------------------------------------------------
// Weight preparation: one wavefront per node cuts its row into parts in fragment order and sums its norms; the rest of the
// grid writes the transposed copy that the all-nodes pass reads.
// ---------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) bmu_wide_prep_kernel(const float* __restrict__ W, int K, int D, int kpad, int tiles, int nch,
                                                            const float* __restrict__ centre, char* __restrict__ blob,
                                                            float* __restrict__ norms, float* __restrict__ wt,
                                                            unsigned int* __restrict__ scal, double* __restrict__ qe,
                                                            int32_t* __restrict__ small)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e < 2 && qe) qe[e] = 0.0;
    if (e < 4 && small) small[e] = 0;
    const int node_groups = tiles * kWTile / 4;               // workgroups that take four nodes each
    if ((int)blockIdx.x >= node_groups) {
        const int64_t t = (int64_t)(blockIdx.x - node_groups) * 256 + threadIdx.x;
        if (t < (int64_t)D * kpad) {
            const int f = (int)(t / kpad), k = (int)(t - (int64_t)f * kpad);
            wt[t] = k < K ? W[(size_t)k * D + f] : 0.0f;
        }
        return;
    }
    __shared__ float most[4][3];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 4 + wave;
    double nrm = 0.0;
    float lo2 = 0.0f, rest2 = 0.0f;
    for (int o = lane; o < nch * 4; o += 64) {
        float v[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int f0 = 8 * o + 4 * h, start = f0 < D - 4 ? f0 : D - 4, shift = f0 - start;    // own elements: >= shift
            float4 w4 = {0.f, 0.f, 0.f, 0.f}, c4 = w4;
            if (k < K) {
                w4 = load4(W + (size_t)k * D + start);
                c4 = load4(centre + start);
            }
            v[4 * h + 0] = shift <= 0 ? w4.x - c4.x : 0.0f;
            v[4 * h + 1] = shift <= 1 ? w4.y - c4.y : 0.0f;
            v[4 * h + 2] = shift <= 2 ? w4.z - c4.z : 0.0f;
            v[4 * h + 3] = shift <= 3 ? w4.w - c4.w : 0.0f;
        }
        bf16x8 hi, lo;
        cut8(v, hi, lo, lo2);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            nrm += (double)v[t] * (double)v[t];
            const float left = (v[t] - (float)hi[t]) - (float)lo[t];
            rest2 = fmaf(left, left, rest2);
        }
        const int chunk = o >> 2, kb = (o >> 1) & 1, g = o & 1;
        char* frag = blob + ((size_t)(k / kWTile) * nch + chunk) * kWBuf + (size_t)((((k % kWTile) >> 5) * 2 + kb) * 2) * 1024 +
                     (g * 32 + (k & 31)) * 16;
        *reinterpret_cast<bf16x8*>(frag) = hi;
        *reinterpret_cast<bf16x8*>(frag + 1024) = lo;
    }
    nrm = wave_sum(nrm);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        lo2 += __shfl_xor(lo2, o);
        rest2 += __shfl_xor(rest2, o);
    }
    if (lane == 0) {
        const float nh = (float)(-0.5 * nrm);
        norms[k] = (k < K && nh > kSplitPadNorm) ? nh : kSplitPadNorm;
        float up = (float)nrm;
        if ((double)up < nrm) up = nextafterf(up, INFINITY);
        most[wave][0] = k < K ? up : 0.0f;
        most[wave][1] = lo2;
        most[wave][2] = rest2;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const int t = threadIdx.x;
        const float m = fmaxf(fmaxf(most[0][t], most[1][t]), fmaxf(most[2][t], most[3][t]));
        if (m > 0.0f) atomicMax(&scal[t == 0 ? 0 : kScalLo + t - 1], __float_as_uint(m));
    }
}

// ---------------------------------------------------------------------------------------------------------
// The tiles.  CAND: the samples are the entries of the re-decision list, and every node that reaches the entry's cut is
// appended to the sample's record (rare: an atomic each); the scores are those of the first pass bit for bit.
// ---------------------------------------------------------------------------------------------------------
template <bool CAND>
__device__ __forceinline__ void wide_tile(const BmuArgs& a, const WideArgs& p, int64_t tile, int split, int64_t total, char* lds)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 1, ws = wave >> 1;               // which node blocks (alternating), which 64 samples
    const int j = lane & 31, g = lane >> 5;
    const int t_lo = split * p.per_split;
    const int t_hi = t_lo + p.per_split < p.tiles ? t_lo + p.per_split : p.tiles;
    const int nch = p.nch, nq = (t_hi - t_lo) * nch;
    if (nq <= 0) return;                                    // (whole workgroup)
    char* const bufA = lds;
    char* const bufB = lds + 2 * kWBuf;
    float* const state = reinterpret_cast<float*>(lds + 4 * kWBuf) + wave * (kWState * 64) + lane;
    float* const nbuf = reinterpret_cast<float*>(lds + 4 * kWBuf) + kWThreads * kWState;
    const unsigned ldsA = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) char*)bufA);

    // ---- the samples this thread brings in: two rows, eight features (an octet) of each per chunk
    const int oct = tid & 3;
    const float* xrow[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        int64_t i = tile * kWTile + (tid >> 2) + 128 * it;
        i = i < total ? i : total - 1;
        if constexpr (CAND) i = (int64_t)a.recheck[i];
        xrow[it] = a.X + (a.idx ? (int64_t)a.idx[i] : i) * a.ldx;
    }
    float xs[2] = {0.f, 0.f}, left2[2] = {0.f, 0.f};
    float4 xr[2][2];
    auto load_item = [&](int it, int ch) {
        const int f0 = ch * kWChunk + oct * 8;
        xr[it][0] = load4(xrow[it] + (f0 < a.D - 4 ? f0 : a.D - 4));
        xr[it][1] = load4(xrow[it] + (f0 + 4 < a.D - 4 ? f0 + 4 : a.D - 4));
    };
    float4 cen[2];
    auto load_centre = [&](int ch) {
        const int f0 = ch * kWChunk + oct * 8;
        cen[0] = load4(a.centre + (f0 < a.D - 4 ? f0 : a.D - 4));
        cen[1] = load4(a.centre + (f0 + 4 < a.D - 4 ? f0 + 4 : a.D - 4));
    };
    // centred, cut, written to buffer `buf`: fragment [sample block][kb][hi | lo], lane slot 32 g + (sample ^ 2 octet) so that
    // eight neighbouring lanes (two samples, four octets) hit different banks
    auto convert_item = [&](int it, int ch, int buf, bool norms) {
        float v[8] = {xr[it][0].x - cen[0].x, xr[it][0].y - cen[0].y, xr[it][0].z - cen[0].z, xr[it][0].w - cen[0].w,
                      xr[it][1].x - cen[1].x, xr[it][1].y - cen[1].y, xr[it][1].z - cen[1].z, xr[it][1].w - cen[1].w};
        const int f0 = ch * kWChunk + oct * 8;
        if (ch == nch - 1) {                                // windows shifted back at the end of the row: own elements only
            const int s0 = f0 - (a.D - 4), s1 = s0 + 4;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                v[t] = t >= s0 ? v[t] : 0.0f;
                v[4 + t] = t >= s1 ? v[4 + t] : 0.0f;
            }
        }
        bf16x8 hi, lo;
        if (!CAND && norms) {
            cut8(v, hi, lo, left2[it]);
#pragma unroll
            for (int t = 0; t < 8; ++t) xs[it] = fmaf(v[t], v[t], xs[it]);
        } else {
            cut8(v, hi, lo);
        }
        const int s = (tid >> 2) + 128 * it;
        char* frag = bufB + buf * kWBuf + ((s >> 5) * 4 + (oct >> 1) * 2) * 1024 + ((oct & 1) * 32 + ((s & 31) ^ (2 * oct))) * 16;
        *reinterpret_cast<bf16x8*>(frag) = hi;
        *reinterpret_cast<bf16x8*>(frag + 1024) = lo;
    };
    // chunk ch of node tile t into buffer `buf`: every wavefront 4 KB
    auto load_weights = [&](int t, int ch, int buf) {
        const char* from = p.blob + ((size_t)t * nch + ch) * kWBuf + wave * 4096 + lane * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) lds_load16(from + q * 1024, ldsA + buf * kWBuf + wave * 4096 + q * 1024);
    };

    // ---- running state per lane, sample block and row parity (CAND: none): best, runner-up, where the best came from
    float cut[2];
    int64_t sample[2];
    if constexpr (CAND) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            const int64_t e = tile * kWTile + ws * 64 + sb * 32 + j;
            cut[sb] = e < total ? a.cutv[e] : NAN;          // no score compares >= NaN
            sample[sb] = (int64_t)a.recheck[e < total ? e : total - 1];
        }
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            state[(3 * c + 0) * 64] = -INFINITY;
            state[(3 * c + 1) * 64] = -INFINITY;
            state[(3 * c + 2) * 64] = 0.0f;
        }
    }

    floatx16 acc[4][2];
    // the scores of node block nb of tile t: as bmu_split_tile's fold, two classes (row parity) per lane; together with the
    // lane halves and the two wavefronts of a sample, neighbouring nodes fall into eight classes
    auto fold = [&](int nb, int t) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
            if constexpr (CAND) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (acc[nb][sb][r] >= cut[sb]) {
                        const unsigned id = (unsigned)(t * kWTile + (2 * nb + wn) * 32 + 8 * (r >> 2) + 4 * g + (r & 3));
                        uint32_t* rec = p.record + sample[sb] * kWRecord;
                        const unsigned at = atomicAdd(rec, 1u);
                        if (at < (unsigned)kWIds) reinterpret_cast<uint16_t*>(rec + 1)[at] = (uint16_t)id;
                    }
            } else {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    float* st = state + (sb * 2 + c) * 3 * 64;
                    float best = st[0], second = st[64];
                    const float before = best;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r0 = 4 * q + c, r1 = r0 + 2;
                        const float v1 = __uint_as_float((__float_as_uint(acc[nb][sb][r0]) & 0xfffffff8u) | (unsigned)(r0 >> 1));
                        const float v2 = __uint_as_float((__float_as_uint(acc[nb][sb][r1]) & 0xfffffff8u) | (unsigned)(r1 >> 1));
                        const float mid = __builtin_amdgcn_fmed3f(best, v1, v2);
                        best = vmax3(best, v1, v2);
                        second = vmax(second, mid);
                    }
                    st[0] = best;
                    st[64] = second;
                    if (best > before) st[128] = __int_as_float(4 * t + nb);
                }
            }
        }
    };
    // blocks of a tile that hold any node at all
    auto blocks_of = [&](int t) {
        const int left = (a.K - t * kWTile + 31) >> 5;
        return left < 8 ? left : 8;
    };

    // ---- first chunk, and the second one's samples on their way
    load_weights(t_lo, 0, 0);
    load_centre(0);
    load_item(0, 0);
    load_item(1, 0);
    if (tid < kWTile) nbuf[tid] = p.norms[t_lo * kWTile + tid];
    convert_item(0, 0, 0, true);
    convert_item(1, 0, 0, true);
    load_item(0, nch > 1 ? 1 : 0);
    load_item(1, nch > 1 ? 1 : 0);
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    int t = t_lo, ch = 0;                       // of chunk q
    for (int q = 0; q < nq; ++q) {
        const int buf = q & 1;
        int ch1 = ch + 1, t1 = t;               // of chunk q + 1
        if (ch1 == nch) {
            ch1 = 0;
            ++t1;
        }
        const int ch2 = ch1 + 1 == nch ? 0 : ch1 + 1;
        const bool more = q + 1 < nq;
        const bool new_tile = more && ch1 == 0;
        float norm_next = 0.0f;
        // (the last iteration requests its own chunk's successor nowhere: its buffers stay unused)
        if (more) load_weights(t1, ch1, buf ^ 1);
        if (new_tile && tid < kWTile) norm_next = p.norms[t1 * kWTile + tid];
        load_centre(ch1);
        const char* fa = bufA + buf * kWBuf + wn * 4096 + lane * 16;
        const char* fb = bufB + buf * kWBuf + ws * 8192;
        bf16x8 xh[2][2], xl[2][2];
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const char* f = fb + kb * 2048 + (g * 32 + (j ^ (4 * kb + 2 * g))) * 16;
#pragma unroll
            for (int sb = 0; sb < 2; ++sb) {
                xh[sb][kb] = *reinterpret_cast<const bf16x8*>(f + sb * 4096);
                xl[sb][kb] = *reinterpret_cast<const bf16x8*>(f + sb * 4096 + 1024);
            }
        }
        const int blocks = blocks_of(t);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) {
            const bool live = 2 * nb + wn < blocks;         // (a block of padding nodes is left out)
            if (live) {
                const char* f = fa + nb * 8192;
                bf16x8 wh[2], wl[2];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    wh[kb] = *reinterpret_cast<const bf16x8*>(f + kb * 2048);
                    wl[kb] = *reinterpret_cast<const bf16x8*>(f + kb * 2048 + 1024);
                }
                floatx16 part[2];
#pragma unroll
                for (int sb = 0; sb < 2; ++sb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) part[sb][r] = 0.0f;
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb) part[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh[kb], xl[sb][kb], part[sb], 0, 0, 0);
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb) part[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl[kb], xh[sb][kb], part[sb], 0, 0, 0);
                }
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int sb = 0; sb < 2; ++sb) part[sb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh[kb], xh[sb][kb], part[sb], 0, 0, 0);
                if (ch == 0) {
                    // the previous tile's scores are folded beside these MFMAs, then the accumulators start at -|w|^2 / 2
                    if (q > 0) fold(nb, t - 1);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const float4 n4 = *reinterpret_cast<const float4*>(nbuf + (2 * nb + wn) * 32 + 8 * u + 4 * g);
#pragma unroll
                        for (int sb = 0; sb < 2; ++sb) {
                            acc[nb][sb][4 * u + 0] = n4.x;
                            acc[nb][sb][4 * u + 1] = n4.y;
                            acc[nb][sb][4 * u + 2] = n4.z;
                            acc[nb][sb][4 * u + 3] = n4.w;
                        }
                    }
                }
#pragma unroll
                for (int sb = 0; sb < 2; ++sb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[nb][sb][r] += part[sb][r];
            } else if (ch == 0 && q > 0) {
                fold(nb, t - 1);                            // (the last tile only: its predecessor's blocks were whole)
            }
            // the next chunk's samples, a quarter of the way on: theirs are the loads of the iteration before
            if (nb == 1 || nb == 2) {
                const int it = nb - 1;
                if (more) convert_item(it, ch1, buf ^ 1, q + 1 < nch);
                load_item(it, ch2);
            }
        }
        if (ch == nch - 1 && new_tile) {
            // every wavefront has read this tile's norms long ago (chunk 0, nch >= 3 chunks and as many barriers back)
            if (tid < kWTile) nbuf[tid] = norm_next;
        }
        // the weights' chunk is complete (the four loads behind it are the samples' of the chunk after next), and so are
        // the LDS writes
        asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        t = t1;
        ch = ch1;
    }
    {
        const int blocks = blocks_of(t_hi - 1);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
            if (2 * nb + wn < blocks) fold(nb, t_hi - 1);
    }
    if constexpr (CAND) return;

    // ---- norms of the samples (the first split's workgroup has them as well as any)
    if (split == 0) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            // four lanes hold a sample's octets; the first two octets of a chunk are in the accumulator of both large MFMAs
            float s = xs[it], w = (oct < 2 ? 4.0f : 1.0f) * xs[it], l = left2[it];
            s += __shfl_xor(s, 1);
            w += __shfl_xor(w, 1);
            l += __shfl_xor(l, 1);
            s += __shfl_xor(s, 2);
            w += __shfl_xor(w, 2);
            l += __shfl_xor(l, 2);
            const int64_t i = tile * kWTile + (tid >> 2) + 128 * it;
            if (oct == 0 && i < total) p.norm[i] = make_float4(s, w, l, 0.0f);
        }
    }
    // ---- a sample's eight class winners of this workgroup
    __syncthreads();
    if (tid < kWTile) {
        const int64_t i = tile * kWTile + tid;
        const float* base = reinterpret_cast<const float*>(lds + 4 * kWBuf);
        BestFour best(-INFINITY);
#pragma unroll
        for (int wn1 = 0; wn1 < 2; ++wn1)
#pragma unroll
            for (int g1 = 0; g1 < 2; ++g1)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float* st = base + (2 * (tid >> 6) + wn1) * (kWState * 64) + ((((tid >> 5) & 1) * 2 + c) * 3) * 64 +
                                      g1 * 32 + (tid & 31);
                    const float v = st[0];
                    const int where = __float_as_int(st[128]);
                    const int r = 2 * (int)(__float_as_uint(v) & 7u) + c;
                    best.others = fmaxf(best.others, st[64]);
                    best.add(v, (where >> 2) * kWTile + (2 * (where & 3) + wn1) * 32 + 8 * (r >> 2) + 4 * g1 + (r & 3));
                }
        if (i < total) best.write(p, split, i, 1.0f);
    }
}

// The splits of a sample tile get workgroup numbers 8 apart: they run on the same XCD at about the same time, and its L2
// serves the rows to all but the first.
__global__ void __launch_bounds__(kWThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_wide_split_kernel(const BmuArgs a, const WideArgs p)
{
    extern __shared__ float4 wide_lds[];
    const int64_t blk = blockIdx.x / (8 * p.splits);
    const int within = (int)(blockIdx.x % (8 * p.splits));
    const int64_t tile = blk * 8 + within % 8;
    if (tile * kWTile >= a.m) return;
    wide_tile<false>(a, p, tile, within / 8, a.m, reinterpret_cast<char*>(wide_lds));
}

// a fixed grid walks the (tile of the list, node tile) units: a short list still spreads over the chip
__global__ void __launch_bounds__(kWThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) bmu_wide_split_cand_kernel(const BmuArgs a, const WideArgs p)
{
    extern __shared__ float4 wide_lds[];
    const unsigned int count = a.scal[a.slot];
    if (count <= p.cand_min) return;
    WideArgs one = p;
    one.per_split = 1;
    const int64_t units = ((int64_t)count + kWTile - 1) / kWTile * p.tiles;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        wide_tile<true>(a, one, u / p.tiles, (int)(u % p.tiles), (int64_t)count, reinterpret_cast<char*>(wide_lds));
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------------
// Join: the winner over the splits, the sample's error bound, and the lists.
// ---------------------------------------------------------------------------------------------------------
// Threads of a workgroup: each takes one atomic on the lists' lengths, about 10 ns after one another (10^6 samples by 256s: 33 to 55 us, by
// 1024s 18); few samples spread over more units by 256s (5000 with sixteen splits: 5 us and 12).
constexpr int kJoinThreads = 1024;
static int join_threads(int64_t m) { return m >= 256 * (int64_t)kJoinThreads ? kJoinThreads : 256; }

template <bool PARTS>
__global__ void __launch_bounds__(kJoinThreads) bmu_wide_join_kernel(const BmuArgs a, const WideArgs p)
{
    __shared__ unsigned int wave_base[2][kJoinThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + tid;
    const int waves = blockDim.x / 64;
    const bool live = i < a.m;
    bool close = false, open = false, near = false;
    float cut = 0.0f;
    if (live) {
        float best = -INFINITY, second = -INFINITY;
        int node = 0;
        const int splits = i < p.tail_row ? p.splits : p.tail_splits;
        for (int s0 = 0; s0 < splits; s0 += 4) {                 // (four loads under way)
            float4 r4[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) r4[u] = p.best[p.result(s0 + u < splits ? s0 + u : s0, i)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (s0 + u >= splits) break;
                const float4 r = r4[u];
                const bool up = r.x > best;
                second = fmaxf(fmaxf(second, up ? best : r.x), fmaxf(r.y, r.z));
                node = up ? __float_as_int(r.w) : node;
                best = up ? r.x : best;
            }
        }
        node = (node >= 0 && node < a.K) ? node : a.K - 1;       // (only padding or non-finite scores get here)
        const float4 n = p.norm[i];
        // The error of a score (as bmu_split_tile): what the cut drops, from the norms of the parts (a second part leaves at most
        // 2^-8 of what the first one left: eight significant bits; summing those squares as well takes registers that the tile
        // does not have, 1.88 -> 2.00 ms at 10^6 x 200); a chunk's small products
        // in the accumulator of four MFMAs, its large ones in two and one (the weighted norm), each charged sixteen
        // roundings of 2^-24 whatever the order of its additions; one rounding per chunk's addition to the tile's
        // accumulators; six units for the centrings and -|w|^2 / 2.
        constexpr float unit = 5.9604645e-08f;
        auto root = [](float v) { return __builtin_amdgcn_sqrtf(v); };      // within a unit in the last place
        const float wmax2 = __uint_as_float(a.scal[0]), wmax = root(wmax2 + kSquaresFloor) * 1.00001f;
        float nx, err_w, err_0, err_n;
        if constexpr (PARTS) {
            nx = n.x;
            err_w = n.y;
            err_0 = n.z;
            err_n = 0.5f * 8.0f * unit;
        } else {
            const float lo_w = root(__uint_as_float(a.scal[kScalLo]) + kSquaresFloor) * 1.001f, rest_w = root(__uint_as_float(a.scal[kScalLo + 1]) + kSquaresFloor) * 1.001f;
            // (four float32 sums of 8 nch squares each, added up: short of their size by one rounding a square at most, half of that in
            // the root; 1 + 2^-13 at D = 16384)
            const float grown = 1.0001f + (float)p.nch * (4.1f * unit);
            nx = root(n.x + kSquaresFloor) * grown;
            const float nl = root(n.z + kSquaresFloor) * grown;
            const float add = (float)(p.nch + 1) * 1.016f;
            err_w = nl * (1.0078125f / 256.0f + 65.28f * unit) + root(n.y + kSquaresFloor) * (grown * 16.256f * unit) + nx * ((6.0f + add) * unit);
            err_0 = nl * lo_w * 1.0078125f + nx * (rest_w * 1.0078125f + lo_w * (65.28f * unit));
            err_n = 0.5f * (6.0f + add) * unit;
        }
        const float wn = -2.0f * p.norms[node];
        const float wb = fminf(root(wn + kSquaresFloor) * 1.00001f, wmax);
        const float err_b = err_w * wb + err_0 + err_n * wb * wb;
        const float bits = fabsf(best) * (1.01f * 1.9073486e-06f);          // two scores' position bits
        const float far2 = fmaxf(nx * nx * 1.00001f - 2.0f * best, 0.0f) * 1.00001f + 2.0f * (err_b + bits);
        const float wo = fminf((nx + root(far2)) * 1.0001f, wmax);          // norm of any node as near as the winner
        const float bound = err_b + err_w * wo + err_0 + err_n * wo * wo + bits + kSquaresFloor;
        close = a.K > 1 && !((best - second) > bound);
        cut = best - bound;
        a.bmu[i] = node;
        if (a.qe) {
            // the statistic n_recheck: best two scores inside a band of fixed relative width, as in bmu_split_tile
            const float rel = 2.0f * (3.0f * 3.8146973e-06f * 1.0078125f + (float)(196 + (a.D + 63) / 64 + 1) * unit) + 12.0f * unit;
            near = close || (a.K > 1 && !((best - second) > ((PARTS ? nx : root(n.x)) * wmax + 0.5f * wmax2) * rel));
        }
        if (close) {
            uint32_t* rec = p.record + i * kWRecord;
            uint16_t* ids = reinterpret_cast<uint16_t*>(rec + 1);
            int hits = 0;
            open = a.K > 65536 || !(cut == cut);
            for (int s0 = 0; s0 < splits && !open; s0 += 4) {    // (one after the other: 10^5 x 2000, whose last rows have sixteen pieces, 20.1 us for 16.5)
                float4 r4[4];
                uint4 q4[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const size_t at = p.result(s0 + u < splits ? s0 + u : s0, i);
                    r4[u] = p.best[at];
                    q4[u] = p.next[at];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (s0 + u >= splits || open) break;
                    const float4 r = r4[u];
                    const uint4 q = q4[u];
                    if (r.x >= cut && hits < kWIds) ids[hits++] = (uint16_t)__float_as_int(r.w);
                    if (r.y >= cut && hits < kWIds) ids[hits++] = (uint16_t)q.z;
                    if (__uint_as_float(q.x) >= cut && hits < kWIds) ids[hits++] = (uint16_t)(q.z >> 16);
                    if (__uint_as_float(q.y) >= cut && hits < kWIds) ids[hits++] = (uint16_t)q.w;
                    open = open || r.z >= cut || hits >= kWIds;
                }
            }
            rec[0] = open ? 0u : (unsigned)hits;                 // an open sample's record is filled by the candidate pass
        }
    }
    // both lists' entries of this workgroup with one atomic
    const unsigned long long m_open = __ballot(close && open), m_known = __ballot(close && !open);
    const auto below = [&](unsigned long long m) {
        return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
    };
    if (lane == 0) {
        wave_base[0][wave] = (unsigned)__popcll(m_open);
        wave_base[1][wave] = (unsigned)__popcll(m_known);
    }
    __syncthreads();
    if (tid == 0) {
        unsigned int n0 = 0, n1 = 0;
        unsigned int at[2][kJoinThreads / 64];
        for (int w = 0; w < waves; ++w) {
            at[0][w] = n0;
            at[1][w] = n1;
            n0 += wave_base[0][w];
            n1 += wave_base[1][w];
        }
        unsigned long long base = 0ull;
        if (n0 | n1)
            base = atomicAdd(reinterpret_cast<unsigned long long*>(&a.scal[a.slot]), (unsigned long long)n0 | ((unsigned long long)n1 << 32));
        for (int w = 0; w < waves; ++w) {
            wave_base[0][w] = (unsigned int)base + at[0][w];
            wave_base[1][w] = (unsigned int)(base >> 32) + at[1][w];
        }
    }
    __syncthreads();
    if (close && open) {
        const unsigned int at = wave_base[0][wave] + below(m_open);
        a.recheck[at] = (uint32_t)i;
        a.cutv[at] = cut;
    } else if (close) {
        a.recheck_end[-1 - (int64_t)(wave_base[1][wave] + below(m_known))] = (uint32_t)i;
    }
    if (a.qe) group_qe_add(a.qe_part, 0.0, 0.0, near ? 1 : 0);
}

// ---------------------------------------------------------------------------------------------------------
// Direct differences over the recorded candidates of both lists: sixteen lanes per sample, each every sixteenth feature;
// lowest distance, then lowest node index.  Samples without a usable record (more than fourteen candidates, none, or a
// list that the candidate pass did not serve) go to the second list, which the all-nodes pass takes.
// ---------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) bmu_wide_exact_kernel(const BmuArgs a, const WideArgs p)
{
    const unsigned int n_open = a.scal[a.slot], n_known = a.scal[a.slot + 1], count = n_open + n_known;
    const int sub = threadIdx.x & 15;
    constexpr unsigned int per_group = 256 / 16;
    for (unsigned int p0 = blockIdx.x * per_group; p0 < count; p0 += gridDim.x * per_group) {
        const unsigned int q = p0 + (threadIdx.x >> 4);
        const bool live = q < count;
        const unsigned int qc = live ? q : count - 1;
        const int64_t i = qc < n_open ? (int64_t)a.recheck[qc] : (int64_t)a.recheck_end[-1 - (int64_t)(qc - n_open)];
        const uint32_t* rec = p.record + i * kWRecord;
        const uint32_t found = rec[0];
        const int64_t row = a.idx ? (int64_t)a.idx[i] : i;
        const float* xr = a.X + row * a.ldx;
        bool served = found > 0u && found <= (uint32_t)kWIds;
        const int c = served ? (int)found : 0;
        const uint16_t* ids = reinterpret_cast<const uint16_t*>(rec + 1);
        float bd = INFINITY;
        int bk = 0x7fffffff;
        constexpr int kBatch = 2;                  // most samples have two candidates
        for (int t0 = 0; t0 < kWIds; t0 += kBatch) {
            if (__ballot(c > t0) == 0ull) break;
            int node[kBatch];
            float d[kBatch];
#pragma unroll
            for (int tt = 0; tt < kBatch; ++tt) {
                const int k = t0 + tt < c ? (int)ids[t0 + tt] : -1;
                node[tt] = k < a.K ? k : -1;
                d[tt] = 0.0f;
            }
            const float* wr[kBatch];
#pragma unroll
            for (int tt = 0; tt < kBatch; ++tt) wr[tt] = a.W + (size_t)(node[tt] >= 0 ? node[tt] : 0) * a.D;
            // Lane `sub` adds up features sub, sub + 16, ...: the order is part of the result, since it decides which of two nodes gets a sample
            // that lies between them to the last bit.  (By four neighbouring features a lane, sixteen bytes a load, such samples went elsewhere.)
            auto add = [&](int f, auto many) {
                constexpr int U = decltype(many)::value;
                float x[U], w[kBatch][U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    x[u] = xr[f + 16 * u];
#pragma unroll
                    for (int tt = 0; tt < kBatch; ++tt) w[tt][u] = wr[tt][f + 16 * u];
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int tt = 0; tt < kBatch; ++tt) {
                        const float df = x[u] - w[tt][u];
                        d[tt] = fmaf(df, df, d[tt]);
                    }
            };
            int f = sub;
            for (; f - sub + 256 <= a.D; f += 256) add(f, std::integral_constant<int, 16>{});      // (48 loads under way)
            for (; f - sub + 64 <= a.D; f += 64) add(f, std::integral_constant<int, 4>{});
            for (; f < a.D; f += 16) add(f, std::integral_constant<int, 1>{});
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
        if (mine && served) a.bmu[i] = bk;
        list_push(&a.scal[a.slot2], a.recheck2, nullptr, mine && !served, i, 0.0f);
    }
}

// distances to the winners, where they are asked for: direct differences on the values as given, sixteen lanes per sample
__global__ void __launch_bounds__(256) bmu_wide_distance_kernel(const BmuArgs a)
{
    const int sub = threadIdx.x & 15;
    constexpr int per_group = 256 / 16;
    double qs = 0.0, qs2 = 0.0;
    for (int64_t p0 = (int64_t)blockIdx.x * per_group; p0 < a.m; p0 += (int64_t)gridDim.x * per_group) {
        const int64_t i = p0 + (threadIdx.x >> 4);
        const bool live = i < a.m;
        const int64_t ic = live ? i : a.m - 1;
        const float* xr = a.X + (a.idx ? (int64_t)a.idx[ic] : ic) * a.ldx;
        const int k = a.bmu[ic];
        const float* wr = a.W + (size_t)(k >= 0 && k < a.K ? k : 0) * a.D;
        float d = 0.0f;
        const int whole = a.D / 64 * 64;
        for (int f = 4 * sub; f < whole; f += 64) {
            const float4 x = load4(xr + f), w = load4(wr + f);
            const float d0 = x.x - w.x, d1 = x.y - w.y, d2 = x.z - w.z, d3 = x.w - w.w;
            d = fmaf(d0, d0, d);
            d = fmaf(d1, d1, d);
            d = fmaf(d2, d2, d);
            d = fmaf(d3, d3, d);
        }
        for (int f = whole + sub; f < a.D; f += 16) {
            const float df = xr[f] - wr[f];
            d = fmaf(df, df, d);
        }
        d += __shfl_xor(d, 8);
        d += __shfl_xor(d, 4);
        d += __shfl_xor(d, 2);
        d += __shfl_xor(d, 1);
        if (live && sub == 0) {
            if (a.d2) a.d2[i] = d;
            qs += sqrt((double)d);
            qs2 += (double)d;
        }
    }
    if (a.qe) group_qe_add(a.qe_part, qs, qs2);
}

// ---------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------
static size_t tile_blob_bytes(int32_t K, int32_t D)
{
    const size_t tiles = ((size_t)K + kWTile - 1) / kWTile, nch = ((size_t)D + kWChunk - 1) / kWChunk;
    return tiles * nch * kWBuf + tiles * kWTile * sizeof(float);
}

static int tile_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small)
{
    const int tiles = (K + kWTile - 1) / kWTile, nch = (D + kWChunk - 1) / kWChunk;
    char* blob = (char*)prep.stage16;
    float* norms = (float*)(blob + (size_t)tiles * nch * kWBuf);
    const int64_t groups = (int64_t)tiles * kWTile / 4 + ((int64_t)D * prep.kpad + 255) / 256;
    hipLaunchKernelGGL(bmu_wide_prep_kernel, dim3((unsigned)groups), dim3(256), 0, ctx->stream, W, K, D, prep.kpad, tiles, nch,
                       prep.centre, blob, norms, prep.wt, prep.scal, qe, small);
    return check_hip(ctx, hipGetLastError(), "bmu (wide) preparation launch");
}

// Workgroups per sample tile: enough that the compute units are busy to the end.  A unit takes one workgroup at a time
// (LDS), so the time goes with rounds x node tiles per workgroup, plus about half a node tile's chunks for filling the
// pipeline and writing the results.
static void tile_plan(WideArgs& p, int64_t m, int32_t K, int32_t D, int units)
{
    p.tiles = (K + kWTile - 1) / kWTile;
    p.nch = (D + kWChunk - 1) / kWChunk;
    const int64_t tiles_m = (m + kWTile - 1) / kWTile;
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= p.tiles && s <= 16; ++s) {
        const int per = (p.tiles + s - 1) / s;
        if ((p.tiles + per - 1) / per != s) continue;
        const double rounds = (double)((tiles_m * s + units - 1) / units);
        const double cost = rounds * ((double)per * p.nch + 3.0);
        if (s == 1 || cost < best_cost * 0.98) {
            best = s;
            best_cost = cost;
        }
    }
    p.norms = (const float*)(p.blob + (size_t)p.tiles * p.nch * kWBuf);
    p.set_splits(m, best, (p.tiles + best - 1) / best, (tiles_m + 7) / 8 * 8 * best);
}

static int tile_launch(som_ctx* ctx, const BmuArgs& a, const WideArgs& p, bool cand)
{
    if (cand) {
        const int64_t most = (a.m + kWTile - 1) / kWTile * p.tiles;
        hipLaunchKernelGGL(bmu_wide_split_cand_kernel, dim3((unsigned)(most < 256 ? most : 256)), dim3(kWThreads), kWLds, ctx->stream, a, p);
    } else {
        static bool attr_set_dev[kMaxDevices] = {};
        const void* kernels[] = {reinterpret_cast<const void*>(static_cast<void (*)(const BmuArgs, const WideArgs)>(bmu_wide_split_kernel)),
                                 reinterpret_cast<const void*>(static_cast<void (*)(const BmuArgs, const WideArgs)>(bmu_wide_split_cand_kernel))};
        if (int rc = wide_raise_lds(ctx, attr_set_dev, kernels, kWLds)) return rc;
        hipLaunchKernelGGL(bmu_wide_split_kernel, dim3((unsigned)p.grid), dim3(kWThreads), kWLds, ctx->stream, a, p);
    }
    return check_hip(ctx, hipGetLastError(), "bmu (wide, split) launch");
}

int wide_raise_lds(som_ctx* ctx, bool* done, const void* const (&kernels)[2], size_t bytes)
{
    bool& attr_set = done[ctx->device];               // the attribute belongs to the device, not to the process
    if (attr_set) return SOM_OK;
    for (const void* k : kernels)
        if (int rc = check_hip(ctx, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes), "raising the dynamic LDS limit"))
            return rc;
    attr_set = true;
    return SOM_OK;
}

// Which form the rows take.  On 321 to 512 nodes, two tiles of nodes, the tile's time goes with its rounds (128 rows a unit; one that is not full
// counts as one, and its lists as one more) and chunks of 32 features, the other form's with the rows and chunks of 64.  Chunk by chunk a
// round takes 0.77 of what cutting and searching its rows does up to 384 nodes, 0.82 up to 448 and 0.88 up to 512.  Of 166 sizes of more than 28,000
// rows this line takes a form that is slower by more than 2 % in eight, by 9 % at most.  Cut beforehand against the tile, whole search: 324,149 x 270
// on 500 nodes 452 us and 417, 647,957 x 321 on 500 1024 and 880, 127,352 x 450 on 321 287 and 249, 231,917 x 300 on 343 339 and 310; but
// 183,006 x 1024 on 512 733 and 801, 198,610 x 352 on 509 355 and 386, 50,831 x 600 on 400 169 and 200.  On 530 to 1296 nodes 300,000 x 257 457 us and
// 454 up to 804 and 929.
int bmu_wide_form(const som_ctx* ctx, int32_t K, int32_t D, int64_t rows)
{
    if (D <= kHeldFeatures) return kWideHeld;
    if (K <= kCutNodes) return kWideTile;
    if (K > kCutNodesMany) return kWideCut;
    const int64_t units = ctx->units, groups = (rows + kWTile - 1) / kWTile * 2, rounds = (groups + units - 1) / units;
    const double full = (double)rows / (0.5 * kWTile * (double)units);
    const double least = 1.3 - 0.08 * ((K - kCutNodes - 1) / 64);
    return ((double)rounds + 1.0) * ((D + 31) / 32) < least * full * (2 * ((D + 63) / 64)) ? kWideTile : kWideCut;
}

size_t bmu_wide_blob_bytes(int form, int32_t K, int32_t D, int32_t kpad)
{
    switch (form) {
    case kWideHeld: return bmu_held_blob_bytes(kpad, D);
    case kWideCut: return bmu_cut_blob_bytes(K, D);
    default: return tile_blob_bytes(K, D);
    }
}

float* bmu_wide_spread(const BmuPrep& prep, int32_t K, int32_t D)
{
    switch (prep.form) {
    case kWideHeld: return bmu_held_spread(prep, D);
    case kWideCut: return bmu_cut_spread(prep, K, D);
    default: return nullptr;
    }
}

int bmu_wide_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small)
{
    switch (prep.form) {
    case kWideHeld: return bmu_held_prepare(ctx, W, K, D, prep, qe, small);
    case kWideCut: return bmu_cut_prepare(ctx, W, K, D, prep, qe, small);
    default: return tile_prepare(ctx, W, K, D, prep, qe, small);
    }
}

static WideArgs wide_args(som_ctx* ctx, const BmuPrep& prep, int32_t K, int32_t D, int64_t m)
{
    WideArgs p{};
    p.blob = (const char*)prep.stage16;
    p.rows = m;
    const int units = ctx->units;
    switch (prep.form) {
    case kWideHeld: bmu_held_plan(p, prep, m, K, D, units); break;
    case kWideCut: bmu_cut_plan(p, prep, m, K, D, units); break;
    default: tile_plan(p, m, K, D, units); break;
    }
    return p;
}

static int wide_launch(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, const WideArgs& p, bool cand)
{
    switch (prep.form) {
    case kWideHeld: return bmu_held_launch(ctx, prep, a, p, cand);
    case kWideCut: return bmu_cut_launch(ctx, a, p, cand);
    default: return tile_launch(ctx, a, p, cand);
    }
}

// Lists up to this length go to the all-nodes pass at once: a candidate tile takes one pass over its chunks however few entries it has, the
// all-nodes pass K D differences an entry.  (That pass takes 33 us at K D = 200,000 and 110 at 800,000 for any list of up to 256
// entries, a candidate pass of held rows 4 to 15, and of rows cut beforehand 14 us where it takes 48 (300 x 1024) and 76 where it takes 322
// (2000 x 1024): none of their lists is short enough.)
static uint32_t cand_min_for(const BmuPrep& prep, const BmuArgs& a) { return a.K > 65536 ? 0xffffffffu : prep.form != kWideTile ? 0u : 256u; }

// A pass's workspace: per-split winners, norms, candidate records, and the parts of rows cut beforehand with their scales.
static size_t wide_work(WideArgs& p, char* w, const BmuPrep& prep, int32_t D, int64_t m)
{
    size_t at = 0;
    auto take = [&](size_t bytes) {
        char* q = w + at;
        at += (bytes + 255) / 256 * 256;
        return q;
    };
    p.best = (float4*)take(p.results() * sizeof(float4));
    p.norm = (float4*)take((size_t)m * sizeof(float4));
    p.record = (uint32_t*)take((size_t)m * kWRecord * sizeof(uint32_t));
    p.next = (uint4*)take(p.results() * sizeof(uint4));
    if (prep.form == kWideCut) {
        p.scales = (float*)take(bmu_cut_scales_bytes(D, m));
        p.cut = take(bmu_cut_parts_bytes(D, m));
    }
    return at;
}

size_t bmu_wide_work_bytes(som_ctx* ctx, const BmuPrep& prep, int32_t K, int32_t D, int64_t m)
{
    WideArgs p = wide_args(ctx, prep, K, D, m);
    return wide_work(p, nullptr, prep, D, m);
}

// most rows of a pass: some hundred bytes a sample, and the parts of rows cut beforehand
int64_t bmu_wide_pass_rows(const BmuPrep& prep, int32_t D)
{
    const int64_t most = (int64_t)1 << 24;
    if (prep.form != kWideCut) return most;
    const int64_t rows = bmu_cut_pass_rows(D);
    return rows < most ? rows : most;
}

int bmu_wide_run(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, void* work)
{
    WideArgs p = wide_args(ctx, prep, a.K, a.D, a.m);
    wide_work(p, (char*)work, prep, a.D, a.m);
    p.cand_min = cand_min_for(prep, a);
    if (int rc = wide_launch(ctx, prep, a, p, false)) return rc;
    const int per_join = join_threads(a.m);
    const dim3 join_grid((unsigned)((a.m + per_join - 1) / per_join)), join_block(per_join);
    if (prep.form == kWideTile)
        hipLaunchKernelGGL(bmu_wide_join_kernel<false>, join_grid, join_block, 0, ctx->stream, a, p);
    else
        hipLaunchKernelGGL(bmu_wide_join_kernel<true>, join_grid, join_block, 0, ctx->stream, a, p);
    return check_hip(ctx, hipGetLastError(), "bmu (wide, split) join launch");
}

// the re-decision (K > 1): candidate pass and direct differences; what is left over is on the second list
int bmu_wide_recheck(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, void* work)
{
    WideArgs p = wide_args(ctx, prep, a.K, a.D, a.m);
    wide_work(p, (char*)work, prep, a.D, a.m);
    p.cand_min = cand_min_for(prep, a);
    if (int rc = wide_launch(ctx, prep, a, p, true)) return rc;
    const int64_t groups = (a.m + 15) / 16;
    hipLaunchKernelGGL(bmu_wide_exact_kernel, dim3((unsigned)(groups < 2048 ? groups : 2048)), dim3(256), 0, ctx->stream, a, p);
    return check_hip(ctx, hipGetLastError(), "bmu (wide, split) candidate-distance launch");
}

int bmu_wide_distances(som_ctx* ctx, const BmuArgs& a)
{
    const int64_t groups = (a.m + 15) / 16;
    hipLaunchKernelGGL(bmu_wide_distance_kernel, dim3((unsigned)(groups < 2048 ? groups : 2048)), dim3(256), 0, ctx->stream, a);
    return check_hip(ctx, hipGetLastError(), "bmu (wide, split) distance launch");
}

} // namespace som
