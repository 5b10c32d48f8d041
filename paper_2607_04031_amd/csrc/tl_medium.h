// Row-adaptive GEMM for medium row counts (tl_medium.hip): parameters and
// configurations.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "tl_internal.h"

namespace tl {

struct MediumParams {
    const uint16_t* A = nullptr;
    const uint8_t* W = nullptr;
    void* C = nullptr;
    unsigned long long* fetch = nullptr;
    int N = 0, K = 0;        // N: columns of C (gated launches: I, of 2I weight rows)
    int64_t strip_bytes = 0;
    int log2_br = 0, log2_bc = 0, log2_G = 0;
    int bc_mask = 0;
    bool out_bf16 = false;
    int n_tiles = 0;         // column tiles
    // load weights that no other workgroup reads non-temporally (only where a
    // K step ends where a line of a weight row does)
    bool w_stream = false;
    // one weight (num_groups 0): total_rows rows in one tile, K split split_k
    // ways (> 1: fp32 partials at ws, ws_stride floats apart)
    int split_k = 1;
    float* ws = nullptr;
    int64_t ws_stride = 0;
    // groups: as tl_gemm_grouped
    const int* offsets = nullptr;
    const int* token_ids = nullptr;
    int num_groups = 0;
    int64_t group_stride = 0;
    int a_rows = 0;
    int total_rows = 0;
};

// Tiles of C (rows x columns) and what a CU holds of them; three weight
// stages, one (256 columns) or two (128) workgroups per CU.
enum class MediumConfig {
    kWide,         // one weight: 256 x 256, 8 waves
    kNarrow,       // one weight: 128 x 128, 4 waves
    kGroupWide,    // groups: 192 x 256, 8 waves
    kGroupNarrow   // groups: 128 x 128, 4 waves
};
inline int medium_tile_m(MediumConfig c) { return c == MediumConfig::kWide ? 256 : c == MediumConfig::kGroupWide ? 192 : 128; }
inline int medium_tile_n(MediumConfig c) { return c == MediumConfig::kWide || c == MediumConfig::kGroupWide ? 256 : 128; }

// One launch (by launch_decode, with DecodeLaunch::medium).
struct MediumLaunch {
    MediumParams p;
    int grid;
    MediumConfig cfg;
    bool tile, swiglu;
};

hipError_t launch_medium(const MediumParams& p, int grid, MediumConfig cfg, bool tile, bool swiglu, hipStream_t stream);

}  // namespace tl
