// Internal declarations shared by the translation units of libsom (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>
#include <vector>

#include "som.h"

namespace som {

constexpr int kNodesPerStage = 128;   // nodes of W staged through LDS at a time by the BMU kernel
constexpr int kTops = 8, kTopsKept = 8;         // BmuPrep::tops
constexpr int kMaxStepsResident = 32; // BMU kernel keeps a sample's features in registers up to D = 64

struct BmuPrep {
    float* stage = nullptr;        // [Kpad / 128][nch] blobs: 128 padded weight rows of a chunk, then -|w|^2 / 2
    void* stage16 = nullptr;       // parts of the weights for the split searches (D <= 64: stage rows of bf16 parts; D > 64: bmu_wide_form), else null
    float* wrow = nullptr;         // [K][D] the weights as given in the stages' order (split search for D <= 64)
    int kb = 0;                    // whole 16-feature blocks of a stage16 row
    int tail_r = 0;                // features of the packed tail block behind them (0: none; D <= 64 only)
    float* wt = nullptr;           // [D][Kpad] transposed weights (as given, not centred); split search for D <= 64: nodes in the stages' order
    float* centre = nullptr;       // [D] column means of W; stage rows and sample registers hold values minus this
    // Result words, cleared by every preparation: [0] = bits of max_k |w_k - centre|^2, [3] = total,
    // [4], [5] = length of the second list (samples whose candidate slots overflowed; alternating calls),
    // [12], [13] = length of the list and of the pair list, [14], [15] the next call's; D > 64, bf16 parts: [8], [9] = bits of max_k |w - hi|^2 and
    // |w - hi - lo|^2, half-precision and fp6 parts: [8..10] = of max_k |second part|, |what fp6 leaves of the first|, |of the second|;
    // half-precision and fp6 parts, any D: [11] = the scale
    unsigned int* scal = nullptr;
    // Split search for D <= 64: kTops maxima, found by atomics in [0..], which are zero whenever no call is in
    // progress; the first pass moves them to [kTopsKept..], where later passes read them.  (What a call leaves behind
    // does not depend on which call it is, so a captured call can be replayed.)  Bits of max_k |w_k - centre|^2; with bf16 parts of |w - hi|^2 and
    // |w - hi - lo|^2; with half-precision and fp6 parts, of |second part|, |what fp6 leaves of the first|, |of the second|, for each unit of
    // |w_k| and as they are, and how far the bits of the least |w_k| without a row of its own lie below those of infinity (0: all have one).
    unsigned int* tops = nullptr;
    int kpad = 0, steps = 0, stride = 0;
    int nch = 1;                   // feature chunks of 2 * steps features (1 unless D > 64)
    int form = 0;                  // split searches: SplitForm (D <= 64) or WideForm
    int calls = 0;                 // bmu_run calls served by this preparation (selects the list counter)
};

struct BmuArgs {
    const float* X;
    int64_t ldx;
    const uint32_t* idx;
    int64_t m;
    int32_t D, K, kpad;
    const float* W;          // caller's dense K x D weights (exact distances)
    const float* stage;      // BmuPrep::stage
    int32_t stride;          // BmuPrep::stride (floats per row of the float32 stage)
    const void* stage16;     // BmuPrep::stage16 (null: float32 search)
    int32_t tail_r;          // BmuPrep::tail_r
    int32_t second_only;     // bmu_exact_kernel: serve the second list whatever the first one's length
    const float* wt;         // BmuPrep::wt
    const float* wrow;       // BmuPrep::wrow
    const float* centre;     // BmuPrep::centre
    unsigned int* scal;      // BmuPrep::scal
    const unsigned int* norms;   // split search, D <= 64: the maxima (BmuPrep::tops, or + kTopsKept after the first pass)
    unsigned int* tops;      // first pass of the same: BmuPrep::tops, to be moved; else null
    int32_t slot;            // scal[slot], scal[slot + 1] count this call's list and pair list (12 or 14)
    int64_t full_tiles;      // bmu_kernel: workgroups below this number take full tiles, the others half tiles
    float* cut_all;          // [m] per presented sample: its cut when it is to be re-decided, a NaN otherwise
    uint32_t* recheck;       // [m] sample positions to re-decide (compacted from cut_all by bmu_list_kernel)
    uint32_t* recheck_end;   // end of the recheck array, from which the pair list grows down
    uint32_t* pairs;         // [m][2], on large maps [m][4], per sample on the pair list: up to four (eight) 16-bit rows of the stages, the used ones
                             // in front (0xffff: none)
    // Candidate pass (long lists only): the search is repeated for the listed samples, and every node whose score
    // reaches the sample's cut is noted; direct differences are then taken over those few nodes only.
    float* cutv;             // [m] per list entry: best score minus the rounding bound (half-precision parts of up to 64 features: at the sample's scale)
    ulonglong2* cand;        // [cand_cap][2]: per list entry and half-wavefront, seven 16-bit node ids and their count
    uint32_t* recheck2;      // [cand_cap] samples left to the all-nodes pass (slots overflowed, or no candidate)
    int32_t slot2;           // which of scal[4], scal[5] counts recheck2
    uint32_t cand_min;       // the candidate pass serves list lengths in (cand_min, cand_cap]
    uint32_t cand_cap;
    int32_t* bmu;            // [m], always written
    float* d2;               // may be null
    double* qe;              // [2], accumulated (caller zeroes); may be null
    double* qe_part;         // [kQeSlots][2] partial sums, then [kQeSlots] near ties (zero on entry, zeroed again by qe_finish_kernel)
    bool qe_later;           // the caller adds them up and zeroes them: qe is not written
    int32_t counts_near;     // the search counts the near ties itself (n_recheck); otherwise the list's length is counted
};

constexpr int kQeSlots = 256;
// Times of an epoch's stages for its statistics, noted by the first workgroup of the kernel that a stage begins with (two 64-bit
// ticks of wall_clock64 in som_ctx::small).  An event between two kernels holds the stream up by 4 us: an epoch of
// 250,000 x 37 on 437 nodes took 149 us with three of them and takes 136.
constexpr int kStampWord = 8, kStampStart = 0, kStampUpdate = 1;
__device__ __forceinline__ void stamp(int32_t* small, int which)
{
    if (small && threadIdx.x == 0 && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        reinterpret_cast<unsigned long long*>(small + kStampWord)[which] = wall_clock64();
}
constexpr int kMaxDevices = 64;                 // devices the per-device tables hold
constexpr int kUpdateStaticCells = 65536;       // som_neighborhood_update_static: K * (D + 1) at most
constexpr int kUpdateStaticNodes = 32768;       // and K at most
constexpr int kCandSlots = 8;         // 16-bit places per (list entry, half-wavefront): up to seven node ids and a count

} // namespace som

struct som_ctx {
    int device = 0;
    int units = 256;               // compute units of the device
    hipStream_t stream = nullptr;
    hipStream_t copy_stream = nullptr;
    char err[512] = {0};
    double eta = 1.0, mu = 0.0;    // update rule (som_set_update_rule)
    float* velocity = nullptr;

    // BMU workspaces (grown on demand)
    void* prep_blob = nullptr;
    size_t prep_bytes = 0;
    bool prep_clean = false;       // its maxima (BmuPrep::tops) are zero
    uint32_t* recheck = nullptr;   // one allocation: lists [cap], cuts [cap], per-sample marks or second list [cap], candidate sets
    size_t recheck_cap = 0;
    bool recheck_sets = false;     // the allocation holds the candidate sets
    uint32_t* pairs = nullptr;     // pair ids, by the row: the searches for up to 64 features only, and on small maps half as many
    size_t pairs_bytes = 0;
    int32_t* bmu_ws = nullptr;     // BMU indices of the epoch drivers (one chunk's worth)
    size_t bmu_elems = 0;
    void* acc_blob = nullptr;      // per-workgroup float64 slices + counts of the accumulation pass
    void* parts_blob = nullptr;    // workspace of a pass of the wide split search (D > 64)
    size_t parts_bytes = 0;
    // The last search that memory kept from passes of `asked` rows: how many it held, and what was left of memory then, the workspaces of a
    // pass counted in.
    struct {
        int64_t asked = 0, held = 0;
        int32_t K = 0, D = 0;
        size_t left = 0;
    } scarce;
    size_t acc_bytes = 0;
    void* upd_blob = nullptr;      // influence matrix + split-k partials of the update
    size_t upd_bytes = 0;
    double* upd_static = nullptr;  // this device's fixed update workspace (som_neighborhood_update_static)
    int safeguard = 0;             // SOM_SAFEGUARD_*
    int reproducible = 0;          // prefer the fixed-order accumulation kernel
    int search = 0;                // SOM_SEARCH_*
    double* qe_part = nullptr;     // [kQeSlots][2], then [kQeSlots], zero between calls
    double* small_sums = nullptr;  // small epochs: three sets of per-node sums and counts (som_small.hip)
    size_t small_clean = 0;        // leading cells of set small_turn (0 or 1) that are zero
    int small_turn = 0;
    void* topo_blob = nullptr;     // node distances, adjacency matrix and lists of the topology rebuild
    size_t topo_bytes = 0;
    // epoch-internal accumulators
    double* S = nullptr;
    size_t S_elems = 0;
    unsigned long long* n = nullptr;
    size_t n_elems = 0;
    double* qe = nullptr;          // double[2]
    int32_t* small = nullptr;      // int32[4]: n_guarded, n_empty, spare; from kStampWord on the times of an epoch
    double clock_khz = 1e5;        // rate of the device's wall clock
    void* host_small = nullptr;    // pinned mirror for reading results back
    // streaming
    float* pinned[2] = {nullptr, nullptr};
    float* dchunk[2] = {nullptr, nullptr};
    size_t chunk_elems = 0;
    hipEvent_t ev_copied[2] = {nullptr, nullptr};
    hipEvent_t ev_consumed[2] = {nullptr, nullptr};
    std::vector<hipEvent_t> h2d_events;   // (start, stop) per chunk of a streamed epoch; grown on demand, reused
    // measurement support: event pairs around every launch of the main BMU kernel while profiling is on
    bool profiling = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_events;
    size_t prof_used = 0;
};

namespace som {

int fail(som_ctx* ctx, int code, const char* fmt, ...);
int check_hip(som_ctx* ctx, hipError_t e, const char* what);

// kernels' host launchers (each returns SOM_OK or an error code after recording detail in ctx)
int launch_fill_zero(som_ctx* ctx, void* p, size_t bytes);
// qe (double[2]) and small (int32[4]) are zeroed by the preparation kernel when given
// rows: how many a bmu_run will bring, as far as the caller knows; all: how many its runs bring together
int bmu_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, int64_t rows, int64_t all, BmuPrep* out, double* qe, int32_t* small);
int bmu_run(som_ctx* ctx, BmuPrep& prep, BmuArgs args);
// split search for D > 64 (som_bmu_wide.hip)
int bmu_wide_form(const som_ctx* ctx, int32_t K, int32_t D, int64_t rows);
size_t bmu_wide_blob_bytes(int form, int32_t K, int32_t D, int32_t kpad);
int bmu_wide_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small);
size_t bmu_wide_work_bytes(som_ctx* ctx, const BmuPrep& prep, int32_t K, int32_t D, int64_t m);
int64_t bmu_wide_pass_rows(const BmuPrep& prep, int32_t D);
int bmu_wide_run(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, void* work);
int bmu_wide_recheck(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, void* work);
int bmu_wide_distances(som_ctx* ctx, const BmuArgs& a);
// small calls (som_small.hip): 1 = not a small one, otherwise SOM_OK or an error code
int small_bmu_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, const float* W, int32_t K,
                  int32_t* bmu, float* d2, double* qe);
int small_epoch_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m, float* W, int32_t K,
                    const float* G, double sigma, double eps_h);
int accumulate_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m,
                   const int32_t* bmu, int32_t K, double* S, unsigned long long* n, bool zero_first);
// 1 = shape not served by the MFMA path (caller falls back), otherwise SOM_OK or an error code
int accumulate_mfma_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m,
                        const int32_t* bmu, int32_t K, double* S, unsigned long long* n, bool zero_first);
// 1 = shape not served; stable: fixed order of summation
int accumulate_sort_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m,
                        const int32_t* bmu, int32_t K, double* S, unsigned long long* n, bool zero_first, bool stable);
constexpr int kFMaxSlabs = 16;                  // most slabs of LDS that accumulate_f64_run serves,
constexpr int64_t kFStride = 1 << 22;           // and rows nearer to each other than this many floats
int accumulate_f64_slabs(int32_t K, int32_t D);
int accumulate_f64_run(som_ctx* ctx, const float* X, int32_t D, int64_t ldx, const uint32_t* idx, int64_t m,
                        const int32_t* bmu, int32_t K, double* S, unsigned long long* n, bool zero_first);
int update_run(som_ctx* ctx, const double* S, const unsigned long long* n, const float* G, int32_t K,
               int32_t D, double sigma, double eps_h, float* W, int32_t* small);
int update_static_init(som_ctx* ctx);
int update_static_run(som_ctx* ctx, const double* S, const unsigned long long* n, const float* G, int32_t K,
                      int32_t D, double sigma, double eps_h, float* W, int32_t* small);

} // namespace som
