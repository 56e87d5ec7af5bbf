// What the searches for more than 64 features share (som_bmu_wide.hip, som_bmu_held.hip): a pass's workspace and its join.
#pragma once

#include "som_bmu_common.hpp"

namespace som {

constexpr int kWIds = 14;                         // candidate ids of a record: 4 bytes count, fourteen 16-bit ids
constexpr int kWRecord = 8;                       // 32-bit words of a record
constexpr int kHeldFeatures = 256;                // most features of a row that the wavefronts hold (som_bmu_held.hip)

struct WideArgs {
    const char* blob;        // weights' parts, [node tile][chunk][node block 8][kb 2][hi | lo][64 lanes][8] bf16
    const float* norms;      // [node tiles * 256] -|w|^2 / 2
    int nch, tiles;          // chunks of a row, node tiles
    int splits, per_split;   // workgroups that share a sample tile, node tiles of each
    int64_t rows;            // m of the pass
    float4* best;            // [splits][m] best, second best class winner, highest of all others; id of the best (bits)
    uint32_t* id2;           // [splits][m] id of the second
    float4* norm;            // [m] |x|^2, weighted |x|^2, |x - hi|^2
    uint32_t* record;        // [m][kWRecord] candidates of the listed samples
    uint32_t cand_min;       // lists up to this length go to the all-nodes pass at once
};

// 64 lanes x 16 bytes, from the lanes' own addresses to 1 KB of LDS at offset lds (below 64 KB); counted by vmcnt
__device__ __forceinline__ void lds_load16(const void* from, unsigned lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(from) : "memory", "m0");
}

// rows held in registers (som_bmu_held.hip)
size_t bmu_held_blob_bytes(int32_t kpad, int32_t D);
float* bmu_held_spread(const BmuPrep& prep, int32_t D);
const float* bmu_held_norms(const BmuPrep& prep, int32_t D);
int bmu_held_prepare(som_ctx* ctx, const float* W, int32_t K, int32_t D, const BmuPrep& prep, double* qe, int32_t* small);
int bmu_held_splits(int64_t m, int32_t K, int32_t D, int units);
int bmu_held_launch(som_ctx* ctx, const BmuPrep& prep, const BmuArgs& a, const WideArgs& p, bool cand);

} // namespace som
