// Decode GEMM for 17 <= M <= 64 with activations and weights staged in LDS.
//
// At M = 32 every workgroup of the streaming decode kernel (tl_decode.hip)
// reloads the activations of its K range from L2, as many bytes again as
// half of the weight bytes it streams (at M = 64 on 64-row tiles, as many as
// the weight bytes); those extra L2 -> CU requests, not HBM, limit it.  Here
// one workgroup (8 waves, one per CU) takes 32 T rows of W -- T whole 32-row
// strips of memory tiles -- and one K range, and walks it in 64-wide K steps:
//   * a step's rows of A and W go from memory straight into one of four LDS
//     stages (16 MT + 32 T rows of 128 bytes, 20 - 32 KB), three steps ahead
//     of their use, so 60 - 96 KB per CU are in flight whatever the registers
//     hold, and A crosses L2 -> CU once per 32 T weight rows; one barrier per
//     step;
//   * wave w takes K half w mod 2 of the step and the 16-row subtiles
//     w / 2, w / 2 + 4, ...: MFMA 16x16x32 on operands read from LDS, W rows
//     by one wave pair, A rows by all;
//   * steps alternate over four sets of sums (fp32 chains as short as when
//     each wave owned every eighth step), added at the end, the K halves
//     through LDS in a fixed order; then stored (one K range) or written as a
//     split-K partial for the fixed-order reduce kernel.
// Staging only A (512 columns per barrier) and streaming W through registers,
// one or two steps in flight, took, on the Llama-70B shapes, one MI355X, bf16
// out, M = 32 / 48: QKV 34.9 / 41.8 us -> 31.5 / 32.1, O - / 33.2 -> - / 30.0,
// gate+up 140.2 / - -> 137.0 / -, down 77.7 / 84.9 -> 72.1 / 73.2 (reads of
// the weights: 24 / 19 / 132 / 66 us).  What is left is the split-K reduce
// (4 - 5 us) and the ramp of a launch.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tl_decode_common.h"

namespace tl {
namespace {

constexpr int kLdsWaves = 8;
constexpr int kLdsThreads = 64 * kLdsWaves;
constexpr int kStages = 4;

// 16 bytes per lane from global memory straight into LDS (lane l's land at
// lds + 16 l), non-temporal or not; inline assembly, so the kernel and not
// the compiler waits for them (see tl_prefill.hip).
template <bool NT>
__device__ inline void lds_load16(const uint8_t* base, uint32_t voff, uint8_t* lds) {
    const uint32_t la = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(la)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(la)
                     : "memory", "m0");
#pragma clang diagnostic pop
}

#define TL_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)

template <int T, int MT>
__global__ __launch_bounds__(kLdsThreads) void decode_lds_kernel(DecodeParams p) {
    constexpr int NSUB = 2 * T;                           // 16-row subtiles of W
    constexpr int WROWS = 32 * T, AROWS = 16 * MT;
    constexpr int STAGE = (WROWS + AROWS) * 128;
    constexpr int WLOADS = WROWS / 8, LOADS = (WROWS + AROWS) / 8;   // 8-row loads per step
    constexpr int LPW = (LOADS + kLdsWaves - 1) / kLdsWaves;         // most loads of a wave per step
    constexpr bool EVEN = LOADS % kLdsWaves == 0;                    // else the later waves have one fewer
    constexpr int SPW = (NSUB + 3) / 4;                   // most subtiles of a wave
    constexpr int RED = 4 * SPW * MT * 64 * 16;           // the second K half's sums
    static_assert(kStages * STAGE <= 160 * 1024 && RED <= kStages * STAGE, "LDS budget");
    __shared__ __attribute__((aligned(16))) uint8_t smem[kStages * STAGE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int group = blockIdx.x / p.split_k;
    const int split = blockIdx.x - group * p.split_k;
    // this workgroup's 64-wide K steps: [kt0, kt0 + KT)
    const int kt0 = int(int64_t(p.ksteps) * split / p.split_k);
    const int KT = int(int64_t(p.ksteps) * (split + 1) / p.split_k) - kt0;

    const int n_base = group * WROWS;
    const uint8_t* w0 = p.W + int64_t(n_base >> p.log2_br) * p.strip_bytes;
    const uint8_t* Ab = reinterpret_cast<const uint8_t*>(p.A);
    // load i of the wave: rows 8 (wave + 8 i) .. + 7 of the stage (W rows,
    // then A rows); lane l: row + l / 8, LDS position l % 8, holding the
    // 16-byte chunk XORed by (row / 2) mod 8, so that the 16 rows of an
    // operand read fall in distinct banks.  Rows of A past M repeat row M - 1
    // (their sums are never stored).
    const int lrow = lane >> 3, lpos = lane & 7;
    uint32_t off[LPW];                                    // (the planner keeps 32 T weight rows below 4 GB)
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int ld = wave + kLdsWaves * i, r = 8 * ld + lrow;
        const int c = lpos ^ ((r >> 1) & 7);
        if (ld < WLOADS)
            off[i] = uint32_t(int64_t(r >> p.log2_br) * p.strip_bytes +
                              (int64_t(r & ((1 << p.log2_br) - 1)) << (p.log2_bc + 1)) + w_koff<true>(p, c * 8));
        else
            off[i] = uint32_t(min(r - WROWS, p.M - 1) * p.K + c * 8) * 2u;
    }
    auto issue = [&](int s) {
        uint8_t* st = smem + (s & (kStages - 1)) * STAGE;
        const int k0 = (kt0 + s) * 64;
        const uint8_t* wk = w0 + w_koff<true>(p, k0);
        const uint8_t* ak = Ab + int64_t(k0) * 2;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int ld = wave + kLdsWaves * i;         // uniform
            if (ld < WLOADS) lds_load16<true>(wk, off[i], st + ld * 1024);
            else if (ld < LOADS) lds_load16<false>(ak, off[i], st + ld * 1024);
        }
    };
    const bool fewer = !EVEN && wave >= LOADS % kLdsWaves;           // uniform
    auto wait = [&](auto stages_c) {                     // all but the last 'stages' steps' loads have landed
        constexpr int ST = decltype(stages_c)::value;
        if (fewer) TL_WAIT_VMCNT(ST * (LPW - 1));
        else TL_WAIT_VMCNT(ST * LPW);
    };
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    const int g = lane >> 4, q = lane & 15;
    const int half = wave & 1, rg = wave >> 1;
    const int fc = ((4 * half + g) ^ ((q >> 1) & 7)) << 4;   // operand chunk position in a row
    f32x4 acc[kStages][SPW][MT];
#pragma unroll
    for (int e = 0; e < kStages; ++e)
#pragma unroll
        for (int i = 0; i < SPW; ++i)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[e][i][mt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // step s, stage and set s mod 4 (a compile-time constant)
    auto step = [&](int s, auto set_c) {
        constexpr int SET = decltype(set_c)::value;
        if (s + 2 < KT) wait(std::integral_constant<int, 2>{});
        else if (s + 1 < KT) wait(std::integral_constant<int, 1>{});
        else wait(std::integral_constant<int, 0>{});
        lds_barrier();
        if (s + 3 < KT) issue(s + 3);                    // into the stage step s - 1 read
        const uint8_t* Ws = smem + SET * STAGE + q * 128 + fc;
        const uint8_t* As = Ws + WROWS * 128;
        bf16x8 a[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[mt] = *reinterpret_cast<const bf16x8*>(As + mt * 2048);
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
            const int j = rg + 4 * i;
            if (NSUB % 4 == 0 || j < NSUB) {             // uniform
                const bf16x8 w = *reinterpret_cast<const bf16x8*>(Ws + j * 2048);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    // weights first: a lane holds four consecutive columns of one row of C
                    acc[SET][i][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, a[mt], acc[SET][i][mt], 0, 0, 0);
            }
        }
    };
    std::integral_constant<int, 0> c0;
    std::integral_constant<int, 1> c1;
    std::integral_constant<int, 2> c2;
    std::integral_constant<int, 3> c3;
    for (int s = 0; s < 3 && s < KT; ++s) issue(s);
    int s = 0;
    for (; s + 4 <= KT; s += 4) {
        step(s, c0);
        step(s + 1, c1);
        step(s + 2, c2);
        step(s + 3, c3);
    }
    if (s < KT) step(s, c0);
    if (s + 1 < KT) step(s + 1, c1);
    if (s + 2 < KT) step(s + 2, c2);

    if (p.fetch && threadIdx.x == 0) atomicAdd(p.fetch, (unsigned long long)KT * WROWS * 128ull);

    // ---- the four sets, then the K halves, in a fixed order ----
    lds_barrier();
    f32x4* red = reinterpret_cast<f32x4*>(smem);         // [rg][i][mt][lane]
#pragma unroll
    for (int i = 0; i < SPW; ++i)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int e = 1; e < kStages; ++e) acc[0][i][mt] += acc[e][i][mt];
            if (half == 1) red[((rg * SPW + i) * MT + mt) * 64 + lane] = acc[0][i][mt];
        }
    lds_barrier();
    if (half == 1) return;
    const bool final_out = p.split_k == 1;
    float* part = p.ws + int64_t(split) * p.ws_stride;
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
        const int j = rg + 4 * i;
        if (NSUB % 4 && j >= NSUB) break;                // uniform
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f32x4 v = acc[0][i][mt] + red[((rg * SPW + i) * MT + mt) * 64 + lane];
            const int m = mt * 16 + q, n = n_base + j * 16 + 4 * g;
            if (m < p.M) {
                // N is a multiple of 32: the four columns are aligned
                if (!final_out) {
                    *reinterpret_cast<f32x4*>(part + int64_t(m) * p.N + n) = v;
                } else if (p.out_bf16) {
                    uint2 o;
                    o.x = uint32_t(f32_to_bf16_rne(v[0])) | (uint32_t(f32_to_bf16_rne(v[1])) << 16);
                    o.y = uint32_t(f32_to_bf16_rne(v[2])) | (uint32_t(f32_to_bf16_rne(v[3])) << 16);
                    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.C) + int64_t(m) * p.N + n) = o;
                } else {
                    *reinterpret_cast<f32x4*>(static_cast<float*>(p.C) + int64_t(m) * p.N + n) = v;
                }
            }
        }
    }
}

template <int T>
hipError_t launch_t(const DecodeParams& p, int grid, hipStream_t stream) {
    if (p.M > 32) {
        if constexpr (T <= 4) {
            hipLaunchKernelGGL((decode_lds_kernel<T, 4>), dim3(grid), dim3(kLdsThreads), 0, stream, p);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL((decode_lds_kernel<T, 2>), dim3(grid), dim3(kLdsThreads), 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_lds_decode(const DecodeParams& p, int tiles_per_wg, int grid, hipStream_t stream) {
    switch (tiles_per_wg) {
        case 4: return launch_t<4>(p, grid, stream);
        case 5: return launch_t<5>(p, grid, stream);
        case 6: return launch_t<6>(p, grid, stream);
        case 7: return launch_t<7>(p, grid, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tl
