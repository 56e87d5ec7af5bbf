// Neighbourhood-weighted batch update in float64 (the normalised update U_j / H_j after Eq. 4, with the
// per-sample sums of Eq. 3 grouped by best-matching unit):
//     Num_j = sum_k h(G[k][j]) S_k,   Den_j = sum_k h(G[k][j]) n_k,   h(g) = exp(-g^2 / (2 sigma^2)),
//     w_j <- Num_j / Den_j  where Den_j >= eps_h, otherwise w_j stays.
// The contraction Num = H^T S (with n as one more column of S) is a dense K x K . K x (D + 1) product in float64:
// it runs on v_mfma_f64_16x16x4_f64.
//   1. contract_kernel     one wavefront = 16, 32 or 64 updated nodes x up to 64 columns x a quarter of a part of the k range; for
//                          D + 1 <= 64 the influences h = exp(-G^2 / 2 sigma^2) are computed in the wavefront right
//                          where the MFMA needs them (each one is needed exactly once), otherwise influence_kernel
//                          writes them out first and the wavefronts of the column slabs read them;
//   2. finish_kernel       adds the parts' partials in a fixed order, applies the threshold, writes W, counts.
#include "som_internal.hpp"

#include <math.h>
#include <type_traits>

#include <mutex>

namespace som {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// Parts of the k range: the four wavefronts of a workgroup take a quarter each and add their results in LDS, and up to
// kSplitK workgroups share a block of updated nodes where those alone leave the chip idle (their partials are stored, then
// summed in order).  With sixteen stored partials whatever the shape, the partials were most of the traffic: 262 MB each way
// at K = 1024, D = 2000 (207 + 53 us for contraction and finish there, 153 to 173 + 7 without; 228 + 28 -> 96 + 5 us at K = 4096, D = 50).
constexpr int kSplitK = 8;

// The shape of a contraction.  Two wavefronts for every SIMD, so that one's loads and exponentials run beside the other's MFMAs:
// 4 per block of nodes and 64 columns, more parts where those are too few.  (One for every SIMD: K = 4096, D = 50 150 us, 100 with
// two; K = 1024, D = 50 17.5, 12.6; K = 437, D = 37 8.8, 6: all with the library's exponential.)
// Several column blocks: as many nodes a wavefront as leave that many.  S comes straight from L2, 512 bytes for each float64 MFMA and block of
// sixteen nodes: with one block L2 is what bounds it, four read it a quarter as often.  Whole update, one block, two, four: K = 1024
// D = 500 66, 48, 44 us, D = 1000 85, 85, 71, D = 2000 122, 120, 116; K = 400 D = 500 24, 26, 26, D = 1000 30, 29, 35, D = 2000 43, 40, 41;
// K = 256 D = 1000 18.5, 21, 24.  (With the masks of ragged ends on every operand, as one block had them before, K = 1024 D = 500 60,
// D = 2000 161; the matrix pipe alone would take 54.)
struct UpdateShape {
    int jt, blocks_j, blocks_c, splits;
};
static UpdateShape update_shape(int K, int D)
{
    UpdateShape u;
    u.blocks_c = (D + 1 + 63) / 64;
    auto blocks_of = [&](int jt) { return (int64_t)((K + 16 * jt - 1) / (16 * jt)) * u.blocks_c; };
    if (u.blocks_c > 1) u.jt = K >= 1024 && blocks_of(4) >= 100 ? 4 : K >= 400 && blocks_of(2) >= 128 ? 2 : 1;
    else u.jt = K >= 2048 ? 2 : 1;
    u.blocks_j = (K + 16 * u.jt - 1) / (16 * u.jt);
    const int64_t blocks = (int64_t)u.blocks_j * u.blocks_c;
    u.splits = blocks >= 512 ? 1 : blocks >= 256 ? 2 : blocks >= 128 ? 4 : kSplitK;
    return u;
}

// shift[j] = min over occupied nodes k of G[k][j]^2 (+inf when there is none): 16 columns per workgroup, every 64th row a thread,
// eight loads under way.  A chain of loads is all there is: with 64 columns and runs of K / 16 rows, whose branches on n[k] kept
// the loads apart, 12.8 us at K = 400, 4.6 now.
__global__ void __launch_bounds__(1024) shift_kernel(const float* __restrict__ G, const unsigned long long* __restrict__ n,
                                                     int K, double* __restrict__ shift, int32_t* __restrict__ stamps)
{
    stamp(stamps, kStampUpdate);
    __shared__ double low[16][16];
    const int l = threadIdx.x & 15, seg = threadIdx.x >> 4, wave = threadIdx.x >> 6;
    const int j = blockIdx.x * 16 + l, jc = j < K ? j : K - 1;
    double m = INFINITY;
    for (int k0 = seg; k0 < K; k0 += 8 * 64) {
        float g[8];
        unsigned long long on[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int k = k0 + 64 * t < K ? k0 + 64 * t : k0;
            g[t] = G[(size_t)k * K + jc];
            on[t] = n[k];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const double g2 = (double)g[t] * (double)g[t];
            m = on[t] != 0ull && g2 < m ? g2 : m;
        }
    }
#pragma unroll
    for (int o = 16; o < 64; o <<= 1) {
        const double other = __shfl_xor(m, o);
        m = other < m ? other : m;
    }
    if ((threadIdx.x & 48) == 0) low[wave][l] = m;
    __syncthreads();
    if (seg == 0 && j < K) {
#pragma unroll
        for (int q = 1; q < 16; ++q) m = low[q][l] < m ? low[q][l] : m;
        shift[j] = m;
    }
}

// exp(x) for x <= 0 (any other x gives some value, NaN gives NaN), to less than one unit in the last place (0.949 the largest error of
// 1.5 * 10^8 arguments against quadruple precision): x = n ln 2 + r, |r| <= ln 2 / 2, and
// 1 + r + r^2 q(r), q interpolated at ten Chebyshev nodes (error 3e-18).  Without a branch and with its constants in scalar registers: the
// library's took some sixty instructions and three branches for 24, and branches keep a batch's loads and MFMAs apart.
// Contraction of K = 4096, D = 50, sixteen million of them: 92 us with the library's, 70 with these.
__device__ __forceinline__ double exp_below(double x)
{
    double c9 = 0x1.af38a9b0ec855p-26, c8 = 0x1.289185613a3d6p-22, c7 = 0x1.71de0dae63bb3p-19, c6 = 0x1.a019b90d2ae7ap-16,
           c5 = 0x1.a01a01a7c41d5p-13, c4 = 0x1.6c16c1788bd90p-10, c3 = 0x1.11111111109b3p-7, c2 = 0x1.5555555553d63p-5,
           c1 = 0x1.5555555555556p-3, c0 = 0x1.0000000000001p-1, log2e = 0x1.71547652b82fep+0, ln2_hi = 0x1.62e42fefa0000p-1,
           ln2_lo = 0x1.cf79abc9e3b3ap-40;
    asm("" : "+s"(c8), "+s"(c7), "+s"(c6), "+s"(c5), "+s"(c4), "+s"(c3), "+s"(c2), "+s"(c1), "+s"(c0));
    asm("" : "+s"(log2e), "+s"(ln2_hi), "+s"(ln2_lo), "+s"(c9));
    x = x < -1100.0 ? -1100.0 : x;                            // (zero from -746 on)
    const double n = __builtin_rint(x * log2e);
    const double r = fma(-n, ln2_lo, fma(-n, ln2_hi, x));
    double q = fma(c9, r, c8);
    q = fma(q, r, c7);
    q = fma(q, r, c6);
    q = fma(q, r, c5);
    q = fma(q, r, c4);
    q = fma(q, r, c3);
    q = fma(q, r, c2);
    q = fma(q, r, c1);
    q = fma(q, r, c0);
    q = fma(fma(q, r, 1.0), r, 1.0);
    return __builtin_amdgcn_ldexp(q, (int)n);
}

// h = exp(-(g^2 - shift_j) / 2 sigma^2); with a shift only occupied nodes k contribute (their exponent is <= 0)
__device__ __forceinline__ double influence_of(double gd, double inv2s2, double shift_j, bool occupied)
{
    double h = exp_below(-(gd * gd - shift_j) * inv2s2);
    asm("" : "+v"(h));                                        // (formed for every lane: the compiler would branch around it otherwise)
    return (isinf(gd) || isinf(shift_j) || !occupied) ? 0.0 : h;
}

__global__ void __launch_bounds__(256) influence_kernel(const float* __restrict__ G, int K, double inv2s2,
                                                        const double* __restrict__ shift,
                                                        const unsigned long long* __restrict__ n, double* __restrict__ H, int32_t* __restrict__ stamps)
{
    stamp(stamps, kStampUpdate);
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (size_t)K * K) return;
    const int k = (int)(e / K), j = (int)(e % K);
    H[e] = influence_of((double)G[e], inv2s2, shift ? shift[j] : 0.0, !shift || n[k] != 0ull);
}

// grid (ceil(K / (16 JT)), ceil((D + 1) / 64), splits), 4 wavefronts per workgroup, a quarter of the workgroup's k range each.
// MFMA operands (16 x 16 x 4, float64): lane l supplies A[i = l % 16][k = l / 16] = h[k][j0 + i] and
// B[k = l / 16][c = l % 16] = S[k][c0 + c] (column D is n); its register r receives row l / 16 + 4 r, column l % 16.
// JT: blocks of sixteen updated nodes per wavefront.
template <bool FUSED, int JT>
__global__ void __launch_bounds__(256, 2) contract_kernel(const float* __restrict__ G, const double* __restrict__ H,
                                                       double inv2s2, const double* __restrict__ shift,
                                                       const double* __restrict__ S,
                                                       const unsigned long long* __restrict__ n, int K, int D,
                                                       double* __restrict__ part, int32_t* __restrict__ stamps)
{
    stamp(stamps, kStampUpdate);
    __shared__ double sums[4][4][4][64];               // [wavefront][column block][register][lane]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j0 = blockIdx.x * 16 * JT, c0 = blockIdx.y * 64;
    const int slices = gridDim.z * 4, z = blockIdx.z * 4 + wave;
    const int kper = ((K + slices * 4 - 1) / (slices * 4)) * 4;
    const int k_lo = z * kper;
    const int k_hi = (k_lo + kper < K) ? k_lo + kper : K;
    const int li = lane & 15, lk = lane >> 4;
    doublex4 acc[JT][4];
    int jc[JT];
    double shift_j[JT];
#pragma unroll
    for (int q = 0; q < JT; ++q) {
        const int j = j0 + 16 * q + li;
        jc[q] = j < K ? j : K - 1;
        shift_j[q] = (FUSED && shift) ? shift[jc[q]] : 0.0;
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[q][t] = doublex4{0.0, 0.0, 0.0, 0.0};
    }
    // kBatch k-steps at a time, the next batch's loads under way during the exponentials and MFMAs of the one in hand.  (Twice as many steps
    // with their loads in front of them: K = 1024, D = 2000 93 us, 79 this way; K = 437, D = 37 5.4 and 4.7; K = 1024, D = 50 9.6 and 10.3, the
    // one size of these that loses, and by less than the others gain: one form for all.)
    constexpr int kBatch = FUSED ? 4 : JT == 4 ? 2 : 4;
    struct Batch {
        float g[FUSED ? JT : 1][kBatch];
        double h[FUSED ? 1 : JT][kBatch];
        double s[kBatch][4];
        unsigned long long count[kBatch];
    };
    // (inner: all columns are of S.  Rows and columns behind the last are formed and not stored.)
    auto load = [&](int kb, Batch& b, auto inner) {
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
            const int k = kb + 4 * s + lk;
            const int kc = k < K ? k : K - 1;                 // clamped row: the loads are unconditional
#pragma unroll
            for (int q = 0; q < JT; ++q) {
                if constexpr (FUSED) b.g[q][s] = G[(size_t)kc * K + jc[q]];
                else b.h[q][s] = H[(size_t)kc * K + jc[q]];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = c0 + 16 * t + li;
                b.s[s][t] = S[(size_t)kc * D + (inner || c < D ? c : D - 1)];
            }
            // (every lane loads the count and one of sixteen takes it: loads of those lanes alone were a branch each between the others)
            if (!inner) b.count[s] = n[kc];
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto use = [&](int kb, Batch& b, auto whole, auto inner) {
#pragma unroll
        for (int s = 0; s < kBatch; ++s) {
            if (!whole && kb + 4 * s >= k_hi) continue;
            const int k = kb + 4 * s + lk;
            const bool occupied = !(FUSED && shift) || b.count[s] != 0ull;       // (FUSED: one block of columns, the last one)
            if (!inner) {
                const double cd = (double)b.count[s];
#pragma unroll
                for (int t = 0; t < 4; ++t) b.s[s][t] = c0 + 16 * t + li == D ? cd : b.s[s][t];
            }
#pragma unroll
            for (int q = 0; q < JT; ++q) {
                const bool in = whole || k < k_hi;
                double h;
                if constexpr (FUSED) h = in ? influence_of((double)b.g[q][s], inv2s2, shift_j[q], occupied) : 0.0;
                else h = in ? b.h[q][s] : 0.0;
#pragma unroll
                for (int t = 0; t < 4; ++t) acc[q][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(h, in ? b.s[s][t] : 0.0, acc[q][t], 0, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // (the steps that a small map's last batch has not are left out; among whole batches the same branches would keep loads and MFMAs apart)
    auto all = [&](auto inner) {
        constexpr int STEP = 4 * kBatch;
        Batch one, two;
        int kb = k_lo;
        if (kb < k_hi) load(kb, one, inner);
        for (; kb + 2 * STEP <= k_hi; kb += 2 * STEP) {
            load(kb + STEP, two, inner);
            use(kb, one, std::true_type{}, inner);
            load(kb + 2 * STEP, one, inner);
            use(kb + STEP, two, std::true_type{}, inner);
        }
        if (kb + STEP <= k_hi) {
            load(kb + STEP, two, inner);
            use(kb, one, std::true_type{}, inner);
            if (kb + STEP < k_hi) use(kb + STEP, two, std::false_type{}, inner);
        } else if (kb < k_hi) {
            use(kb, one, std::false_type{}, inner);
        }
    };
    if (c0 + 64 <= D) all(std::true_type{});
    else all(std::false_type{});
#pragma unroll
    for (int q = 0; q < JT; ++q) {
        if (q > 0) __syncthreads();
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) sums[wave][t][r][lane] = acc[q][t][r];
        __syncthreads();
        const int c = c0 + 16 * wave + li;                     // wavefront w adds up column block w
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int jr = j0 + 16 * q + lk + 4 * r;
            const double v = ((sums[0][wave][r][lane] + sums[1][wave][r][lane]) + sums[2][wave][r][lane]) + sums[3][wave][r][lane];
            if (jr < K && c <= D) part[((size_t)blockIdx.z * K + jr) * (D + 1) + c] = v;
        }
    }
}

// plain = true: w <- Num / Den (eta = 1, no momentum);  otherwise delta = eta (Num / Den - w) + mu v, w += delta
template <int SPLITS>
__global__ void __launch_bounds__(256) finish_kernel(const double* __restrict__ part,
                                                     const unsigned long long* __restrict__ n, int K, int D,
                                                     double eps_h, bool plain, double eta, double mu,
                                                     float* __restrict__ V, float* __restrict__ W,
                                                     int32_t* __restrict__ small)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    const size_t stride = (size_t)K * (D + 1);
    if (small && e < K) {
        // guarded and empty nodes: one atomic per wavefront and counter (one per node, all on two words, took 20 us of a
        // 4096-node map's update)
        double den = 0.0;
#pragma unroll
        for (int z = 0; z < SPLITS; ++z) den += part[z * stride + (size_t)e * (D + 1) + D];
        const unsigned long long guarded = __ballot(!(den >= eps_h)), empty = __ballot(n[e] == 0ull);
        if ((threadIdx.x & 63) == 0) {
            if (guarded) atomicAdd(&small[0], (int)__popcll(guarded));
            if (empty) atomicAdd(&small[1], (int)__popcll(empty));
        }
    }
    if (e >= K * D) return;
    const int j = e / D, d = e % D;
    const double* row = part + (size_t)j * (D + 1);
    double num = 0.0, den = 0.0;
#pragma unroll
    for (int z = 0; z < SPLITS; ++z) {
        num += row[z * stride + d];
        den += row[z * stride + D];
    }
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

// the three launches of one update on the given workspaces: H [K*K] (only when D + 1 > 64), part [splits*K*(D+1)],
// shift [K] (only with the shifted-exponent safeguard)
static int update_launch(som_ctx* ctx, double* H, double* part, double* shift_ws, const double* S,
                         const unsigned long long* n, const float* G, int32_t K, int32_t D, double sigma, double eps_h,
                         float* W, int32_t* small)
{
    const size_t h_elems = (size_t)K * K;
    const double inv2s2 = 1.0 / (2.0 * sigma * sigma);
    const UpdateShape u = update_shape(K, D);
    const int jt = u.jt, splits = u.splits;
    const dim3 grid(u.blocks_j, u.blocks_c, splits);
    double* shift = nullptr;
    int32_t* stamps = small;                                  // the first launch notes the time
    if (ctx->safeguard == SOM_SAFEGUARD_SHIFT) {
        shift = shift_ws;
        hipLaunchKernelGGL(shift_kernel, dim3((K + 15) / 16), dim3(1024), 0, ctx->stream, G, n, K, shift, stamps);
        stamps = nullptr;
        if (int rc = check_hip(ctx, hipGetLastError(), "exponent shift launch")) return rc;
    }
    if (grid.y == 1) {
        auto kern = jt == 2 ? contract_kernel<true, 2> : contract_kernel<true, 1>;
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, ctx->stream, G, (const double*)nullptr, inv2s2, (const double*)shift, S, n, K, D,
                           part, stamps);
    } else {
        hipLaunchKernelGGL(influence_kernel, dim3((unsigned)((h_elems + 255) / 256)), dim3(256), 0, ctx->stream, G, K, inv2s2,
                           (const double*)shift, n, H, stamps);
        if (int rc = check_hip(ctx, hipGetLastError(), "influence kernel launch")) return rc;
        auto kern = jt == 4 ? contract_kernel<false, 4> : jt == 2 ? contract_kernel<false, 2> : contract_kernel<false, 1>;
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, ctx->stream, G, (const double*)H, inv2s2, (const double*)nullptr, S, n, K, D, part, (int32_t*)nullptr);
    }
    if (int rc = check_hip(ctx, hipGetLastError(), "contraction kernel launch")) return rc;
    const bool plain = ctx->eta == 1.0 && ctx->mu == 0.0;
    auto finish = splits == 1 ? finish_kernel<1> : splits == 2 ? finish_kernel<2> : splits == 4 ? finish_kernel<4> : finish_kernel<kSplitK>;
    hipLaunchKernelGGL(finish, dim3((K * D + 255) / 256), dim3(256), 0, ctx->stream, part, n, K, D, eps_h, plain,
                       ctx->eta, ctx->mu, ctx->velocity, W, small);
    return check_hip(ctx, hipGetLastError(), "update finish launch");
}

int update_run(som_ctx* ctx, const double* S, const unsigned long long* n, const float* G, int32_t K, int32_t D,
               double sigma, double eps_h, float* W, int32_t* small)
{
    const size_t h_elems = (size_t)K * K;
    const size_t parts = (size_t)update_shape(K, D).splits * K * (D + 1);
    const size_t need = (h_elems + parts + K) * sizeof(double);
    if (need > ctx->upd_bytes) {
        if (ctx->upd_blob) {
            if (int rc = check_hip(ctx, hipStreamSynchronize(ctx->stream), "sync before workspace growth")) return rc;
            (void)hipFree(ctx->upd_blob);
            ctx->upd_blob = nullptr;
            ctx->upd_bytes = 0;
        }
        if (hipMalloc(&ctx->upd_blob, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(ctx, SOM_ENOMEM, "cannot allocate %zu bytes for the update workspace", need);
        }
        ctx->upd_bytes = need;
    }
    double* H = (double*)ctx->upd_blob;
    double* part = H + h_elems;
    return update_launch(ctx, H, part, part + parts, S, n, G, K, D, sigma, eps_h, W, small);
}

// ---------------------------------------------------------------------------------------------------------
// The same update for callers that cannot allocate (som_neighborhood_update_static): the split-k partials and the
// exponent shifts live in a fixed device array instead of a grown workspace.  One array per GPU, shared by every
// call on that GPU and holding the last call's contents; every cell a call reads it has written first (the
// contraction writes every node and column of the partials that its launch has, the finish kernel reads those, the shift
// kernel writes every node), so nothing needs clearing.  Host code never uses the array's name as an address: the device address is looked up once per device.
// ---------------------------------------------------------------------------------------------------------
static __device__ __align__(256) double scratch[(size_t)kSplitK * kUpdateStaticCells + kUpdateStaticNodes];

static std::mutex g_scratch_mutex;
static double* g_scratch_ptr[kMaxDevices] = {};     // per device: its own copy of the array, at its own address

// called by som_create with the context's device current
int update_static_init(som_ctx* ctx)
{
    if (ctx->device < 0 || ctx->device >= kMaxDevices) return SOM_OK;   // the static entry point reports it when used
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[ctx->device]) {
        void* p = nullptr;
        if (int rc = check_hip(ctx, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "looking up the static update workspace")) return rc;
        g_scratch_ptr[ctx->device] = (double*)p;
    }
    ctx->upd_static = g_scratch_ptr[ctx->device];
    return SOM_OK;
}

int update_static_run(som_ctx* ctx, const double* S, const unsigned long long* n, const float* G, int32_t K, int32_t D,
                      double sigma, double eps_h, float* W, int32_t* small)
{
    if (D + 1 > 64 || K > kUpdateStaticNodes || (int64_t)K * (D + 1) > kUpdateStaticCells)
        return fail(ctx, SOM_EINVAL,
                    "som_neighborhood_update_static serves D <= 63, K <= %d and K * (D + 1) <= %d (got K = %d, D = %d)",
                    kUpdateStaticNodes, kUpdateStaticCells, K, D);
    if (!ctx->upd_static) return fail(ctx, SOM_ESTATE, "the static update workspace was not set up on this device");
    double* part = ctx->upd_static;
    return update_launch(ctx, nullptr, part, part + (size_t)kSplitK * kUpdateStaticCells, S, n, G, K, D, sigma, eps_h, W, small);
}

} // namespace som
