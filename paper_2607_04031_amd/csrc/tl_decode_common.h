// Shared by the decode kernels (tl_decode.hip, tl_decode_fp8.hip, tl_lgms.hip):
// kernel parameters and small device helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "tl_internal.h"

namespace tl {

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));


struct DecodeParams {
    const uint16_t* A;
    const uint8_t* W;
    void* C;
    float* ws;
    unsigned long long* fetch;
    int M, N, K;
    int split_k;
    int steps_per_unit;      // 64-element steps per split unit
    int units;               // ceil(K / k_unit)
    int ksteps;              // ceil(K / 64): 64-element K steps
    int kfull;               // K / 64: steps wholly inside K (a last partial step is masked)
    int64_t ws_stride;       // floats between two splits' partials (M * N rounded up to 4)
    int64_t strip_bytes;     // br * Kp * s (TILE) -- bytes per strip of br rows, Kp = K padded to bc
    int log2_br, log2_bc, log2_G;
    int bc_mask;
    bool out_bf16;
    int log2_fetch;          // block-granular emulation on a row-major weight: log2(G)
    int64_t w_bytes;         // N * K * 2
    // grouped (one launch over many weights, e.g. MoE experts)
    const int* offsets;      // [groups + 1] output-row offsets of the groups
    const int* token_ids;    // A row of each output row, or nullptr (identity)
    int tiles_per_group;     // N / tile_n
    int64_t group_stride;    // bytes between consecutive groups' weights
    int a_rows;              // rows of A; token ids outside [0, a_rows) read zeros
    int total_rows;          // rows of C; group offsets are clamped to [0, total_rows]
    const float* scales;     // FP8 weights: per-output-channel scale [N], or nullptr (1)
    unsigned* arrive;        // K splits summed inside the launch (kernels with FUSE): one arrival counter per tile, else nullptr
    int swiglu_up;           // gated grouped launch: row of the first up row (I); C has N = I columns
    int arrive_clear;        // arrive + arrive_clear: the set of counters to clear for the next such launch
};

__device__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu))  // NaN stays NaN
        return uint16_t((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

__device__ inline void store_out(void* C, int64_t idx, float v, bool out_bf16) {
    if (out_bf16) static_cast<uint16_t*>(C)[idx] = f32_to_bf16_rne(v);
    else static_cast<float*>(C)[idx] = v;
}

// Byte offset of the 8-element chunk starting at (row base, k) of the weight.
template <bool TILE>
__device__ inline int64_t w_koff(const DecodeParams& p, int k) {
    if (TILE) return (int64_t(k >> p.log2_bc) << p.log2_G) + int64_t((k & p.bc_mask) << 1);
    return int64_t(k) << 1;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Value of 'v' held by lane l ^ 8 (DPP row_ror:8 inside each 16-lane row).
__device__ inline bf16x8 swap8(bf16x8 v) {
    i32x4 x = __builtin_bit_cast(i32x4, v), y;
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = __builtin_amdgcn_update_dpp(0, x[i], 0x128, 0xf, 0xf, false);
    return __builtin_bit_cast(bf16x8, y);
}

__device__ inline bf16x8 load_stream(const uint8_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p));
}

// K splits summed inside the launch (p.arrive): every workgroup stores its
// fp32 partial, waits until it is out and counts itself at its tile's counter;
// the workgroup that finds all the others' there sums the tile's partials in
// split order -- the same sums, bit for bit, as splitk_reduce_kernel.  Nobody
// waits for another workgroup.  The splits of a tile run on different XCDs,
// whose L2s are not coherent with each other, so partials are written through
// and read past them (agent scope) instead of writing back a whole L2 at a
// fence.  A counter wraps to zero with its last arrival, in one operation, and
// the launch clears the stream's other set of counters, which the next such
// launch uses: a count that a launch outside the stream's order left behind
// (a replay that overlaps other calls) is gone two such launches later.
__device__ inline void store_partial(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Columns [n0, n0 + COLS) of C (n0 a multiple of 4), after this workgroup's
// partials of them were stored.  Every thread of the workgroup calls it.
template <int COLS, int THREADS>
__device__ inline void splitk_finish(const DecodeParams& p, int tile, int n0) {
    __shared__ unsigned arrived;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wave's partials are out
    __syncthreads();
    if (threadIdx.x == 0) arrived = atomicInc(p.arrive + tile * kArriveStride, unsigned(p.split_k) - 1);
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < kArriveTiles; i += THREADS)
            __hip_atomic_store(p.arrive + p.arrive_clear + i * kArriveStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (arrived != unsigned(p.split_k) - 1) return;     // uniform over the workgroup
    constexpr int kAhead = 8;                           // partials in flight per thread
    if (p.N % 4 == 0) {
        typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
        for (int e = threadIdx.x; e < p.M * (COLS / 4); e += THREADS) {
            const int m = e / (COLS / 4), n = n0 + e % (COLS / 4) * 4;
            if (n >= p.N) continue;
            const int64_t at = int64_t(m) * p.N + n;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            for (int s0 = 0; s0 < p.split_k; s0 += kAhead) {
                u64x2 x[kAhead];
#pragma unroll
                for (int s = 0; s < kAhead; ++s)
                    if (s0 + s < p.split_k) {
                        unsigned long long* src = reinterpret_cast<unsigned long long*>(p.ws + (s0 + s) * p.ws_stride + at);
                        x[s][0] = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        x[s][1] = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                for (int s = 0; s < kAhead; ++s)
                    if (s0 + s < p.split_k) {
                        const f32x4 part = __builtin_bit_cast(f32x4, x[s]);
                        v = s0 + s == 0 ? part : v + part;
                    }
            }
            if (p.out_bf16) {
                uint2 o;
                o.x = uint32_t(f32_to_bf16_rne(v[0])) | (uint32_t(f32_to_bf16_rne(v[1])) << 16);
                o.y = uint32_t(f32_to_bf16_rne(v[2])) | (uint32_t(f32_to_bf16_rne(v[3])) << 16);
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.C) + at) = o;
            } else {
                *reinterpret_cast<f32x4*>(static_cast<float*>(p.C) + at) = v;
            }
        }
    } else {
        for (int e = threadIdx.x; e < p.M * COLS; e += THREADS) {
            const int m = e / COLS, n = n0 + e % COLS;
            if (n >= p.N) continue;
            const int64_t at = int64_t(m) * p.N + n;
            float v = 0.f;
            for (int s0 = 0; s0 < p.split_k; s0 += kAhead) {
                float x[kAhead];
#pragma unroll
                for (int s = 0; s < kAhead; ++s)
                    if (s0 + s < p.split_k)
                        x[s] = __hip_atomic_load(p.ws + (s0 + s) * p.ws_stride + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int s = 0; s < kAhead; ++s)
                    if (s0 + s < p.split_k) v = s0 + s == 0 ? x[s] : v + x[s];
            }
            store_out(p.C, at, v, p.out_bf16);
        }
    }
}

// FP8-weight decode (tl_decode_fp8.hip): launches decode_fp8_kernel for the
// given M tiles, 16-row subtiles per tile, waves and layout.
hipError_t launch_fp8_decode(const DecodeParams& p, int grid, int m_tiles16, int ns, int waves, bool tile,
                             hipStream_t stream);

// Decode over a [K][N] row-major weight (tl_decode_kn.hip): 64-column tiles
// with 4 or 8 waves, or 256-column ones (wide, M <= 32) with 8, p.units 64-row K
// steps split p.split_k ways; block-granular fetch (64-column tiles) when
// p.log2_fetch > 0.
hipError_t launch_kn_decode(const DecodeParams& p, bool wide, int grid, int m_tiles16, int waves, hipStream_t stream);

// Decode through LDS (tl_decode_lds.hip): 17 <= M <= 64, tile-major,
// tiles_per_wg 32-row tiles per workgroup (4..7 for M <= 32, 4 above), the
// p.ksteps 64-wide K steps split p.split_k ways.
hipError_t launch_lds_decode(const DecodeParams& p, int tiles_per_wg, int grid, hipStream_t stream);

}  // namespace tl
