// Row-adaptive GEMM for medium row counts: C = A * W^T with bf16 MFMA 32x32x16
// and fp32 accumulation, W tile-major (or row-major [N][K]), for stacks of
// weights that each serve some tens to some hundreds of rows (the expert
// GEMMs of a mixture-of-experts layer over a prompt or a large decode batch)
// and for one weight at up to 224 rows (K split across workgroups where its
// tiles are fewer than the CUs, fp32 partials summed in split order).
//
// Between decode (16 rows or fewer: read the weights, the rest is free) and
// prefill (MFMA-bound) a call is bound by streaming each weight byte once
// while every byte also feeds a few row blocks' MFMAs; 128 rows per expert
// need about 1500 of the 2800 cycles that a CU's share of HBM takes per K
// step.  So the kernel is built as a stream with the arithmetic under it:
//  - a tile holds all the rows a group usually has (up to 256), so a weight
//    byte is read by one workgroup, and only the 32-row blocks that exist are
//    computed: block b belongs to wave half b mod 2, and the K loop is
//    compiled for each block count;
//  - A (gathered by token id) and W go from memory straight into LDS, W two
//    K steps ahead where the LDS holds three stages, so 32 - 64 KB per CU are
//    in flight whatever the registers hold; one barrier per 64-wide K step;
//  - a wave owns 64 weight rows (gated: 32 gate rows and the 32 up rows of
//    the same columns) and its half's row blocks: 2 + n operand reads per
//    2 n MFMAs;
//  - lanes without a row, or past K, load from a 16-byte zero chunk, so
//    ragged rows, out-of-range token ids and a partial last K step need no
//    masks in the loop.
// Llama-70B gate+up, one MI355X, bf16 out, M = 65 / 96 / 128 / 192: 147 / 161 /
// 177 / 205 us (177 / 185 / 193 / 223 on the kernels of tl_prefill.hip; the
// weight's read takes 132); the planner's comments have the other shapes.
// Qwen-3-30B-A3B experts, one MI355X, both projections, bf16 out: 512 / 1024 /
// 2048 tokens (32 / 64 / 128 rows per expert) 379 / 589 / 1001 us on the
// decode kernel's 64-row passes -> 213 / 230 / 271 us; reading the weights
// once takes 170 us.  Non-temporal weight loads, taken when a group's rows
// fit one tile, are part of that (512 tokens: 228 -> 213 us); with row chunks
// that share the weight they cost (8 groups of 256 rows: 158 -> 165 us), as
// does starting each workgroup at another K step (no gain, the tile's strips
// do not collide in HBM).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "tl_medium.h"

namespace tl {
namespace {

typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ inline uint32_t bf16x2_rne(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, bf16x2_t));
}

// What a lane loads in place of elements that do not exist: rows past the
// tile's last, token ids outside A, columns past K.
__device__ const u32x4 g_zero_chunk = {0u, 0u, 0u, 0u};

// 16 bytes per lane from global memory straight into LDS (lane l's land at
// lds + 16 l); inline assembly, so the kernel and not the compiler waits for
// them (the same instruction and reasons as in tl_prefill.hip).
__device__ inline void lds_load16(const uint8_t* base, uint32_t voff, uint8_t* lds) {
    const uint32_t la = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(la)
                 : "memory", "m0");
#pragma clang diagnostic pop
}
__device__ inline void lds_load16_nt(const uint8_t* base, uint32_t voff, uint8_t* lds) {
    const uint32_t la = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(la)
                 : "memory", "m0");
#pragma clang diagnostic pop
}
__device__ inline void lds_load16_at(const uint8_t* ptr, uint8_t* lds) {
    const uint32_t la = uint32_t(uintptr_t((__attribute__((address_space(3))) void*)lds));
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(ptr), "s"(la)
                 : "memory", "m0");
#pragma clang diagnostic pop
}

#define TL_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)

template <int WN, int MAXB, int WST, bool TILE, bool GROUPED, bool SWIGLU>
__global__ __launch_bounds__(128 * WN) __attribute__((amdgpu_waves_per_eu(2, 2))) void medium_kernel(MediumParams p) {
    constexpr int NWAVES = 2 * WN;
    constexpr int BN = 64 * WN;                  // weight rows per tile
    constexpr int BM = 64 * MAXB;                // most rows of A per tile
    constexpr int A_ST = BM * 128, W_ST = BN * 128;
    constexpr int AI = BM / 8 / NWAVES;          // A loads (8 rows each) per wave and step
    constexpr int WI = BN / 8 / NWAVES;          // W loads per wave and step: 4
    constexpr int LDS = 2 * A_ST + WST * W_ST;
    constexpr int ESTRIDE = 272;                 // epilogue: a row of 64 fp32 + 16 bytes
    static_assert(LDS <= 160 * 1024, "LDS budget");
    static_assert(NWAVES * 32 * ESTRIDE <= LDS, "the epilogue fits in the operand stages");
    static_assert(WI == 4 && AI >= 1, "loads per wave");
    __shared__ __attribute__((aligned(16))) uint8_t smem[LDS];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int half = wave / WN, nq = wave % WN;

    // ---- which rows and columns ----
    int nt, split = 0, row0, rows;               // output rows [row0, row0 + rows)
    const uint8_t* W = p.W;
    if constexpr (GROUPED) {
        // workgroup u runs on XCD u mod 8; the tiles of one slot stay on one
        // XCD (they share rows of A) and the slots in use, a prefix of all
        // slots, are dealt to the XCDs in turn
        const int u = blockIdx.x;
        const int v = u >> 3;
        const int slot = (v / p.n_tiles) * 8 + (u & 7);
        nt = v % p.n_tiles;
        int base = 0, group = -1, chunk = 0, r0 = 0, r1 = 0;
        for (int e0 = 0; e0 < p.num_groups; e0 += 64) {
            const int e = e0 + lane;
            int a = 0, b = 0;
            if (e < p.num_groups) {
                a = min(max(p.offsets[e], 0), p.total_rows);
                b = min(max(p.offsets[e + 1], a), p.total_rows);
            }
            const int nch = (b - a + BM - 1) / BM;
            int incl = nch;
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const int o = __shfl_up(incl, s);
                if (lane >= s) incl += o;
            }
            const unsigned long long hit = __ballot(base + incl > slot);
            if (hit) {
                const int l = __builtin_ctzll(hit);
                group = e0 + l;
                chunk = slot - (base + __shfl(incl, l) - __shfl(nch, l));
                r0 = __shfl(a, l);
                r1 = __shfl(b, l);
                break;
            }
            base += __shfl(incl, 63);
        }
        if (group < 0) return;                   // uniform over the workgroup
        group = __builtin_amdgcn_readfirstlane(group);
        chunk = __builtin_amdgcn_readfirstlane(chunk);
        r0 = __builtin_amdgcn_readfirstlane(r0);
        r1 = __builtin_amdgcn_readfirstlane(r1);
        const int nch = (r1 - r0 + BM - 1) / BM, blocks = (r1 - r0 + 31) / 32;
        const int b0 = int(int64_t(blocks) * chunk / nch), b1 = int(int64_t(blocks) * (chunk + 1) / nch);
        row0 = r0 + b0 * 32;
        rows = min(r0 + b1 * 32, r1) - row0;
        W += int64_t(group) * p.group_stride;
    } else {
        // one weight, all rows in one tile: column tiles, then K splits; each
        // XCD takes a contiguous range (its workgroups share a K range of A)
        const int T = gridDim.x, b = blockIdx.x;
        const int lb = (T % 8 == 0) ? (b % 8) * (T / 8) + b / 8 : b;
        split = lb / p.n_tiles;
        nt = lb - split * p.n_tiles;
        row0 = 0;
        rows = p.total_rows;
    }
    // this workgroup's 64-wide K steps: [kt0, kt0 + KT)
    const int ksteps = (p.K + 63) / 64;
    const int kt0 = GROUPED ? 0 : int(int64_t(ksteps) * split / p.split_k);
    const int KT = GROUPED ? ksteps : int(int64_t(ksteps) * (split + 1) / p.split_k) - kt0;
    const int nblocks = (rows + 31) / 32;

    // ---- per-lane sources ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const uint8_t* Ab = reinterpret_cast<const uint8_t*>(p.A);
    const uint8_t* zero = reinterpret_cast<const uint8_t*>(&g_zero_chunk);
    const uint8_t* aptr[AI];                     // this lane's chunk of the first A step
    uint32_t astep[AI];                          // 128, or 0 where there is no row
    int achunk[AI];                              // k of the chunk inside a step
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int r = 8 * (wave + NWAVES * i) + lrow;
        const int c = lpos ^ ((r >> 1) & 7);
        bool ok = r < rows;
        int src = row0 + r;
        if constexpr (GROUPED) {
            if (p.token_ids) {
                if (ok) src = p.token_ids[src];
                ok = ok && src >= 0 && src < p.a_rows;
            }
        }
        achunk[i] = c * 8;
        aptr[i] = ok ? Ab + (int64_t(src) * p.K + int64_t(kt0) * 64 + c * 8) * 2 : zero;
        astep[i] = ok ? 128u : 0u;
    }
    auto w_koff = [&](int k) -> uint32_t {
        if (TILE) return (uint32_t(k >> p.log2_bc) << p.log2_G) + uint32_t((k & p.bc_mask) << 1);
        return uint32_t(k) << 1;
    };
    const int n_base = SWIGLU ? nt * (BN / 2) : nt * BN;
    // the tile's first weight row as a uniform base, rows as 32-bit offsets
    const int64_t tile_off = TILE ? int64_t(n_base >> p.log2_br) * p.strip_bytes : int64_t(n_base) * p.K * 2;
    const uint8_t* wtile = W + tile_off;
    uint32_t w_row[WI];
    int wchunk[WI];
#pragma unroll
    for (int i = 0; i < WI; ++i) {
        const int r = 8 * (wave + NWAVES * i) + lrow;
        const int c = lpos ^ ((r >> 1) & 7);
        int n;
        if constexpr (SWIGLU) {
            // of each 64 weight rows of the tile, 32 gate rows and the 32
            // up rows of the same columns
            n = min(n_base + (r >> 6) * 32 + (r & 31), p.N - 1) + ((r & 32) ? p.N : 0);
        } else {
            n = min(n_base + r, p.N - 1);
        }
        int64_t off;
        if (TILE) off = int64_t(n >> p.log2_br) * p.strip_bytes + (int64_t(n & ((1 << p.log2_br) - 1)) << (p.log2_bc + 1));
        else off = int64_t(n) * p.K * 2;
        wchunk[i] = c * 8;
        w_row[i] = uint32_t(off - tile_off) + w_koff(c * 8);
    }
    auto issue_a = [&](int s) {
        uint8_t* st = smem + (s & 1) * A_ST;
        const int left = p.K - (kt0 + s) * 64;           // columns of the step inside K
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const int ga = wave + NWAVES * i;
            if (ga * 8 < nblocks * 32) {         // uniform
                const uint8_t* src = left < 64 && achunk[i] >= left ? zero : aptr[i] + uint64_t(uint32_t(s)) * astep[i];
                lds_load16_at(src, st + ga * 1024);
            }
        }
    };
    auto issue_w = [&](int s) {
        uint8_t* st = smem + 2 * A_ST + (WST == 3 ? s % 3 : (s & 1)) * W_ST;
        const int k0 = (kt0 + s) * 64;
        const uint8_t* wk = wtile + w_koff(k0);
        if (k0 + 64 <= p.K && p.w_once) {        // uniform
#pragma unroll
            for (int i = 0; i < WI; ++i) lds_load16_nt(wk, w_row[i], st + (wave + NWAVES * i) * 1024);
        } else if (k0 + 64 <= p.K) {
#pragma unroll
            for (int i = 0; i < WI; ++i) lds_load16(wk, w_row[i], st + (wave + NWAVES * i) * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < WI; ++i)
                lds_load16_at(k0 + wchunk[i] < p.K ? wk + w_row[i] : zero, st + (wave + NWAVES * i) * 1024);
        }
    };
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };

    const int l31 = lane & 31, khalf = lane >> 5;
    const int fsw = (l31 >> 1) & 7;
    // sums of (set, block i, weight half j) at 2 (set blocks + i) + j: with one
    // or two blocks the four 16-wide sub-steps of a K step keep four or two
    // sets, added at the end -- shorter fp32 chains (a sum's rounding error
    // grows with its chain), and MFMAs that do not wait for each other
    f32x16 acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

    issue_a(0);
    issue_w(0);
    if (WST == 3 && KT > 1) issue_w(1);
    // this wave's 32-row blocks: half, half + 2, ... below nblocks
    auto kloop = [&](auto cnt_c) {
        constexpr int CNT = decltype(cnt_c)::value;
        constexpr int SETS = CNT == 1 ? 4 : CNT == 2 ? 2 : 1;
        for (int s = 0; s < KT; ++s) {
            if (WST == 3 && s + 1 < KT) TL_WAIT_VMCNT(WI);
            else TL_WAIT_VMCNT(0);
            lds_barrier();
            if (s + 1 < KT) issue_a(s + 1);
            if (WST == 3) {
                if (s + 2 < KT) issue_w(s + 2);
            } else {
                if (s + 1 < KT) issue_w(s + 1);
            }
            if constexpr (CNT > 0) {
                const uint8_t* As = smem + (s & 1) * A_ST + (half * 32 + l31) * 128;
                const uint8_t* Ws = smem + 2 * A_ST + (WST == 3 ? s % 3 : (s & 1)) * W_ST + (nq * 64 + l31) * 128;
                bf16x8 fa[2][CNT], fb[2][2];
                auto fread = [&](int ss, int buf) {
                    const int c = ((2 * ss + khalf) ^ fsw) << 4;
#pragma unroll
                    for (int j = 0; j < 2; ++j) fb[buf][j] = *reinterpret_cast<const bf16x8*>(Ws + j * 4096 + c);
#pragma unroll
                    for (int i = 0; i < CNT; ++i) fa[buf][i] = *reinterpret_cast<const bf16x8*>(As + i * 8192 + c);
                };
                fread(0, 0);
#pragma unroll
                for (int ss = 0; ss < 4; ++ss) {
                    if (ss < 3) fread(ss + 1, (ss + 1) & 1);
#pragma unroll
                    for (int i = 0; i < CNT; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            // weights first: D rows are columns of C, so a lane
                            // holds runs of four columns of one row
                            acc[2 * (ss % SETS * CNT + i) + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                fb[ss & 1][j], fa[ss & 1][i], acc[2 * (ss % SETS * CNT + i) + j], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int set = 1; set < SETS; ++set)
#pragma unroll
            for (int i = 0; i < 2 * CNT; ++i) acc[i] += acc[2 * CNT * set + i];
    };
    const int cnt = (nblocks - half + 1) / 2;
    switch (cnt) {
        case 0: kloop(std::integral_constant<int, 0>{}); break;
        case 1: kloop(std::integral_constant<int, 1>{}); break;
        case 2: kloop(std::integral_constant<int, (MAXB < 2 ? MAXB : 2)>{}); break;
        case 3: kloop(std::integral_constant<int, (MAXB < 3 ? MAXB : 3)>{}); break;
        default: kloop(std::integral_constant<int, MAXB>{}); break;
    }
    if (p.fetch && t == 0) atomicAdd(p.fetch, (unsigned long long)KT * (unsigned long long)W_ST);

    // ---- epilogue: each wave turns its blocks row-major through its own
    // part of LDS, one 32-row block at a time ----
    lds_barrier();                               // every wave is past its last operand read
    uint8_t* E = smem + wave * 32 * ESTRIDE;
    constexpr int CW = SWIGLU ? 32 : 64;         // output columns per wave
    const int col0 = n_base + nq * CW;
    // one K range of several: its fp32 partial, summed by the split-K reduce
    const bool part = !GROUPED && p.split_k > 1;
    float* F = part ? p.ws + int64_t(split) * p.ws_stride : static_cast<float*>(p.C);
    uint16_t* H = static_cast<uint16_t*>(p.C);
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        if (i >= cnt) break;                     // uniform
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = 8 * g + 4 * khalf;
            if constexpr (SWIGLU) {
                f32x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = acc[2 * i][4 * g + e];
                    h[e] = a / (1.0f + expf(-a)) * acc[2 * i + 1][4 * g + e];
                }
                *reinterpret_cast<f32x4*>(E + l31 * ESTRIDE + c * 4) = h;
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const f32x4 v = {acc[2 * i + j][4 * g], acc[2 * i + j][4 * g + 1], acc[2 * i + j][4 * g + 2], acc[2 * i + j][4 * g + 3]};
                    *reinterpret_cast<f32x4*>(E + l31 * ESTRIDE + (j * 32 + c) * 4) = v;
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
        const int rb = (half + 2 * i) * 32;      // first row of the block in the tile
        if (p.out_bf16 && !part) {
            constexpr int LPR = CW / 8;          // lanes per row, eight columns each
#pragma unroll
            for (int q = 0; q < 32 * LPR / 64; ++q) {
                const int r = q * (64 / LPR) + lane / LPR, c = (lane % LPR) * 8;
                const f32x4 a = *reinterpret_cast<const f32x4*>(E + r * ESTRIDE + c * 4);
                const f32x4 b = *reinterpret_cast<const f32x4*>(E + r * ESTRIDE + c * 4 + 16);
                const int col = col0 + c;
                if (rb + r < rows && col < p.N) {
                    uint16_t* dst = H + int64_t(row0 + rb + r) * p.N + col;
                    const u32x4 o = {bf16x2_rne(a[0], a[1]), bf16x2_rne(a[2], a[3]), bf16x2_rne(b[0], b[1]),
                                     bf16x2_rne(b[2], b[3])};
                    if (col + 8 <= p.N && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
                        *reinterpret_cast<u32x4*>(dst) = o;
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            if (col + e < p.N) dst[e] = uint16_t(o[e >> 1] >> (16 * (e & 1)));
                    }
                }
            }
        } else {
            constexpr int LPR = CW / 4;
#pragma unroll
            for (int q = 0; q < 32 * LPR / 64; ++q) {
                const int r = q * (64 / LPR) + lane / LPR, c = (lane % LPR) * 4;
                const f32x4 a = *reinterpret_cast<const f32x4*>(E + r * ESTRIDE + c * 4);
                const int col = col0 + c;
                if (rb + r < rows && col < p.N) {
                    float* dst = F + int64_t(row0 + rb + r) * p.N + col;
                    if (col + 4 <= p.N && (reinterpret_cast<uintptr_t>(dst) & 15) == 0) {
                        *reinterpret_cast<f32x4*>(dst) = a;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (col + e < p.N) dst[e] = a[e];
                    }
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
    }
}

template <int WN, int MAXB, int WST>
hipError_t launch_c(const MediumParams& p, int grid, bool tile, bool swiglu, hipStream_t stream) {
    const dim3 g(grid), b(128 * WN);
    if (p.num_groups == 0) {
        if (tile) hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, true, false, false>), g, b, 0, stream, p);
        else hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, false, false, false>), g, b, 0, stream, p);
    } else if (swiglu) {
        if (tile) hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, true, true, true>), g, b, 0, stream, p);
        else hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, false, true, true>), g, b, 0, stream, p);
    } else {
        if (tile) hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, true, true, false>), g, b, 0, stream, p);
        else hipLaunchKernelGGL((medium_kernel<WN, MAXB, WST, false, true, false>), g, b, 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_medium(const MediumParams& p, int grid, MediumConfig cfg, bool tile, bool swiglu, hipStream_t stream) {
    switch (cfg) {
        case MediumConfig::kWide: return launch_c<4, 4, 3>(p, grid, tile, swiglu, stream);
        case MediumConfig::kPair192: return launch_c<2, 3, 2>(p, grid, tile, swiglu, stream);
        case MediumConfig::kPair128: return launch_c<2, 2, 3>(p, grid, tile, swiglu, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace tl
