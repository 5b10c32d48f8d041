// Row-adaptive GEMM for medium row counts: C = A * W^T with bf16 MFMA
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
//  - a tile holds all the rows a group usually has (up to 192; one weight:
//    256), so a weight byte is read by one workgroup, and only the 32-row
//    blocks that exist are computed: block b belongs to wave half b mod 2, and
//    the K loop is compiled for each block count.  More rows are cut into
//    chunks of about the same size, whose workgroups run next to each other
//    on one XCD and share the weight in its L2;
//  - A (gathered by token id) and W go from memory straight into LDS, W two
//    K steps ahead, so 32 - 64 KB per CU are
//    in flight whatever the registers hold; one barrier per 64-wide K step;
//  - a wave owns 64 weight rows (gated: 32 gate rows and the 32 up rows of
//    the same columns) and its half's row blocks;
//  - lanes without a row, or past K, load from a 16-byte zero chunk, so
//    ragged rows, out-of-range token ids and a partial last K step need no
//    masks in the loop.
// Sums.  One weight: MFMA 32x32x16 in K order, as in tl_prefill.hip.  Groups:
// the sums of the decode kernel that smaller groups run on, bit for bit -- a
// row's result does not depend on how many rows its group has.  That kernel's
// four waves each sum every fourth K step (MFMA 16x16x32, both halves of a
// step in one chain) and are added in order.  A wave that kept the four sums
// of its tile side by side would need 4 x 96 registers; so it walks the K
// steps in the order 0, 4, 8, ..., 1, 5, 9, ..., 2, ..., 3, ... and keeps the
// sum at hand and the total: 2 x 96, which is what bounds a tile to 192 rows.
// The order costs no time: memory tiles of 4 KB are read whole either way, and
// row-major weights gain (128 experts of 128 rows, both projections: 298 us in K
// order, 269 in this one).  One chain over all of K, on tiles of 256 rows, was
// 3.6e-7 from the exact sums at K = 8192, where this is 2.7e-7, and is faster
// only for groups of 193 - 256 rows (128 experts of 200 rows: 328 us against 383).
// Llama-70B gate+up, one MI355X, bf16 out, M = 65 / 96 / 128 / 192: 147 / 161 /
// 177 / 205 us (177 / 185 / 193 / 223 on the kernels of tl_prefill.hip; the
// weight's read takes 132); the planner's comments have the other shapes.
// Qwen-3-30B-A3B experts, one MI355X, both projections, bf16 out: 512 / 1024 /
// 2048 tokens (32 / 64 / 128 rows per expert) 380 / 586 / 1020 us on the
// decode kernel's 64-row passes -> 212 / 231 / 265 us; reading the weights
// once takes 183 us.  Groups of 200 rows, two chunks: 1493 -> 383 us.
// Non-temporal weight loads, taken when a group's rows fit one tile (and for
// one weight by the rule at its launch, tl_api.cpp), are part of that (512
// tokens: 228 -> 213 us; weights of 2 - 200 MB 0 - 10 %); with row chunks
// that share the weight they cost (8 groups of 256 rows: 158 -> 165 us), and
// with rows of W that are not whole lines, whose ends two K steps share (96 x
// 57701 x 1992 row-major: 71.9 -> 78.2 us with them, 70.3 without), as
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

// Sum of the lanes up to this one (DPP: row shifts, then the last lane of a
// row, and of the first two rows, to those after it), and a lane's value.
__device__ inline unsigned scan64(unsigned v) {
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x111, 0xf, 0xf, true));
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x112, 0xf, 0xf, true));
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x114, 0xf, 0xf, true));
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x118, 0xf, 0xf, true));
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x142, 0xa, 0xf, false));
    v += unsigned(__builtin_amdgcn_update_dpp(0, int(v), 0x143, 0xc, 0xf, false));
    return v;
}
__device__ inline unsigned lane_value(unsigned v, int lane) { return unsigned(__builtin_amdgcn_readlane(int(v), lane)); }

#define TL_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x0F70)

template <int WN, int MAXB, bool TILE, bool GROUPED, bool SWIGLU>
__global__ __launch_bounds__(128 * WN) __attribute__((amdgpu_waves_per_eu(2, 2))) void medium_kernel(MediumParams p) {
    constexpr int NWAVES = 2 * WN;
    constexpr int BN = 64 * WN;                  // weight rows per tile
    constexpr int BM = 64 * MAXB;                // most rows of A per tile
    constexpr int WST = 3;                       // weight stages
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
    // non-temporal weight loads, where no other workgroup reads the tile's weight
    bool w_once = p.w_stream;
    const uint8_t* W = p.W;
    if constexpr (GROUPED) {
        // units in use: group by group, in a group tile by tile, in a tile
        // its chunks of rows; each XCD takes a contiguous range of them
        // (workgroup u runs on XCD u mod 8), so the tiles of a group share its
        // rows of A in one L2, and neighbouring workgroups the weight of a
        // tile.  The first 64 kAhead groups are read once, all at a time.
        constexpr int kAhead = 4;
        auto rows_of = [&](int e, int& a, int& b) -> unsigned {      // chunks of group e
            const int c = min(e, p.num_groups - 1);
            a = min(max(p.offsets[c], 0), p.total_rows);
            b = e < p.num_groups ? min(max(p.offsets[c + 1], a), p.total_rows) : a;
            return unsigned(b - a + BM - 1) / BM;
        };
        int ga[kAhead], gb[kAhead];
        unsigned gn[kAhead], upto[kAhead], mine = 0;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) gn[i] = rows_of(i * 64 + lane, ga[i], gb[i]);
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            upto[i] = i * 64 < p.num_groups ? scan64(gn[i]) : 0u;
            mine += lane_value(upto[i], 63);
        }
        int ra, rb;
        for (int e0 = 64 * kAhead; e0 < p.num_groups; e0 += 64) mine += lane_value(scan64(rows_of(e0 + lane, ra, rb)), 63);
        // (more than the grid holds: offsets out of order)
        if (mine > gridDim.x / unsigned(p.n_tiles)) return;
        const unsigned units = mine * unsigned(p.n_tiles), share = (units + 7) / 8;
        const unsigned at = (blockIdx.x & 7) * share + (blockIdx.x >> 3);
        if ((blockIdx.x >> 3) >= share || at >= units) return;
        const unsigned slot = at / unsigned(p.n_tiles);
        unsigned base = 0, chunks = 0;
        int group = -1, r0 = 0, r1 = 0;
        auto find = [&](int e0, unsigned n, unsigned to, int a, int b) {     // slot among groups e0 .. e0 + 63
            const unsigned long long hit = __ballot(base + to > slot);
            if (!hit) {
                base += lane_value(to, 63);
                return;
            }
            const int l = __builtin_ctzll(hit);
            group = e0 + l;
            chunks = lane_value(n, l);
            base += lane_value(to, l) - chunks;
            r0 = int(lane_value(unsigned(a), l));
            r1 = int(lane_value(unsigned(b), l));
        };
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (group < 0) find(i * 64, gn[i], upto[i], ga[i], gb[i]);
        for (int e0 = 64 * kAhead; e0 < p.num_groups && group < 0; e0 += 64) {
            const unsigned n = rows_of(e0 + lane, ra, rb);
            find(e0, n, scan64(n), ra, rb);
        }
        // (counts of out-of-order offsets can wrap: still a tile and a chunk
        // of this group, or nothing)
        const unsigned unit = at - base * unsigned(p.n_tiles);
        if (group < 0 || chunks < 1 || unit / chunks >= unsigned(p.n_tiles)) return;
        nt = int(unit / chunks);
        const int chunk = int(unit - unsigned(nt) * chunks), blocks = (r1 - r0 + 31) / 32;
        const int b0 = int(int64_t(blocks) * chunk / int(chunks)), b1 = int(int64_t(blocks) * (chunk + 1) / int(chunks));
        row0 = r0 + b0 * 32;
        rows = min(r0 + b1 * 32, r1) - row0;
        w_once = p.w_stream && chunks == 1;
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
    // the step after k in the order of the sums: one by one, or (groups) 0, 4,
    // 8, ..., then 1, 5, 9, ..., then 2, ..., then 3, ...
    auto after = [&](int k) -> int {
        if constexpr (!GROUPED) return k + 1;
        return k + 4 < ksteps ? k + 4 : (k & 3) + 1;
    };

    // ---- per-lane sources ----
    const int lrow = lane >> 3, lpos = lane & 7;
    const uint8_t* Ab = reinterpret_cast<const uint8_t*>(p.A);
    const uint8_t* zero = reinterpret_cast<const uint8_t*>(&g_zero_chunk);
    const uint8_t* aptr[AI];                     // this lane's chunk of K step 0
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
        aptr[i] = ok ? Ab + (int64_t(src) * p.K + c * 8) * 2 : zero;
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
    // K step k into stage s mod the number of stages
    auto issue_a = [&](int k, int s) {
        uint8_t* st = smem + (s & 1) * A_ST;
        const int left = p.K - k * 64;           // columns of the step inside K
#pragma unroll
        for (int i = 0; i < AI; ++i) {
            const int ga = wave + NWAVES * i;
            if (ga * 8 < nblocks * 32) {         // uniform
                const uint8_t* src = left < 64 && achunk[i] >= left ? zero : aptr[i] + uint64_t(uint32_t(k)) * astep[i];
                lds_load16_at(src, st + ga * 1024);
            }
        }
    };
    auto issue_w = [&](int k, int s) {
        uint8_t* st = smem + 2 * A_ST + s % WST * W_ST;
        const int k0 = k * 64;
        const uint8_t* wk = wtile + w_koff(k0);
        if (k0 + 64 <= p.K && w_once) {          // uniform
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

    // the loop over the K steps: a step's loads are issued one (A) and two (W)
    // steps ahead of its MFMAs
    int ka = kt0, kw = kt0;                      // the steps last loaded
    issue_a(ka, 0);
    issue_w(kw, 0);
    if (KT > 1) issue_w(kw = after(kw), 1);
    auto for_steps = [&](auto compute) {
        for (int s = 0; s < KT; ++s) {
            if (s + 1 < KT) TL_WAIT_VMCNT(WI);
            else TL_WAIT_VMCNT(0);
            lds_barrier();
            if (s + 1 < KT) issue_a(ka = after(ka), s + 1);
            if (s + 2 < KT) issue_w(kw = after(kw), s + 2);
            compute(smem + (s & 1) * A_ST, smem + 2 * A_ST + s % WST * W_ST);
        }
    };
    // this wave's 32-row blocks: half, half + 2, ... below nblocks
    const int cnt = (nblocks - half + 1) / 2;
    // weights are the MFMAs' first operand: D rows are columns of C, so a lane
    // holds runs of four columns of one row
    const int l31 = lane & 31, khalf = lane >> 5;
    const int q = lane & 15, g4 = lane >> 4;
    // one weight: MFMA 32x32x16.  Sums of (set, block i, weight half j) at
    // 2 (set blocks + i) + j: with one or two blocks the four 16-wide sub-steps
    // of a K step keep four or two sets, added at the end -- shorter fp32
    // chains (a sum's rounding error grows with its chain), and MFMAs that do
    // not wait for each other
    f32x16 acc[GROUPED ? 1 : 8];
    // groups: MFMA 16x16x32, a set for each of the four classes of steps
    // (mod 4), one after the other: 'part' the class at hand, 'sum' those
    // before it.  [block][16 rows][16 columns]
    f32x4 part[GROUPED ? MAXB : 1][2][4], sum[GROUPED ? MAXB : 1][2][4];
    if constexpr (GROUPED) {
#pragma unroll
        for (int i = 0; i < MAXB; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) sum[i][e >> 2][e & 3] = part[i][e >> 2][e & 3] = f32x4{0.f, 0.f, 0.f, 0.f};
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    }
    auto kloop = [&](auto cnt_c) {
        constexpr int CNT = decltype(cnt_c)::value;
        if constexpr (CNT == 0) {
            for_steps([](const uint8_t*, const uint8_t*) {});
        } else if constexpr (GROUPED) {
            const int fsw = (q >> 1) & 7;
            int k = 0;
            for_steps([&](const uint8_t* A_st, const uint8_t* W_st) {
                const uint8_t* As = A_st + (half * 32 + q) * 128;
                const uint8_t* Ws = W_st + (nq * 64 + q) * 128;
                bf16x8 fa[2][CNT][2], fb[2][4];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int c = ((4 * h + g4) ^ fsw) << 4;
#pragma unroll
                    for (int j = 0; j < 4; ++j) fb[h][j] = *reinterpret_cast<const bf16x8*>(Ws + j * 2048 + c);
#pragma unroll
                    for (int i = 0; i < CNT; ++i)
#pragma unroll
                        for (int m = 0; m < 2; ++m)
                            fa[h][i][m] = *reinterpret_cast<const bf16x8*>(As + i * 8192 + m * 2048 + c);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < CNT; ++i)
#pragma unroll
                        for (int m = 0; m < 2; ++m)
#pragma unroll
                            for (int j = 0; j < 4; ++j)
                                part[i][m][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[h][i][m], part[i][m][j], 0, 0, 0);
                if (k + 4 >= ksteps) {           // the last step of its class
#pragma unroll
                    for (int i = 0; i < CNT; ++i)
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            sum[i][e >> 2][e & 3] += part[i][e >> 2][e & 3];
                            part[i][e >> 2][e & 3] = f32x4{0.f, 0.f, 0.f, 0.f};
                        }
                }
                k = after(k);
            });
        } else {
            constexpr int SETS = CNT == 1 ? 4 : CNT == 2 ? 2 : 1;
            const int fsw = (l31 >> 1) & 7;
            for_steps([&](const uint8_t* A_st, const uint8_t* W_st) {
                const uint8_t* As = A_st + (half * 32 + l31) * 128;
                const uint8_t* Ws = W_st + (nq * 64 + l31) * 128;
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
                            acc[2 * (ss % SETS * CNT + i) + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                fb[ss & 1][j], fa[ss & 1][i], acc[2 * (ss % SETS * CNT + i) + j], 0, 0, 0);
                }
            });
#pragma unroll
            for (int set = 1; set < SETS; ++set)
#pragma unroll
                for (int i = 0; i < 2 * CNT; ++i) acc[i] += acc[2 * CNT * set + i];
        }
    };
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
    const bool partial = !GROUPED && p.split_k > 1;
    float* F = partial ? p.ws + int64_t(split) * p.ws_stride : static_cast<float*>(p.C);
    uint16_t* H = static_cast<uint16_t*>(p.C);
#pragma unroll
    for (int i = 0; i < MAXB; ++i) {
        if (i >= cnt) break;                     // uniform
        if constexpr (GROUPED) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int j = 0; j < (SWIGLU ? 2 : 4); ++j) {
                    f32x4 v = sum[i][m][j];
                    if constexpr (SWIGLU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = v[e] / (1.0f + expf(-v[e])) * sum[i][m][j + 2][e];
                    }
                    *reinterpret_cast<f32x4*>(E + (m * 16 + q) * ESTRIDE + (j * 16 + 4 * g4) * 4) = v;
                }
        } else {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int c = 8 * g + 4 * khalf;
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
        if (p.out_bf16 && !partial) {
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

template <int WN, bool GROUPED, int MAXB, bool SWIGLU = false>
hipError_t launch_c(const MediumParams& p, int grid, bool tile, hipStream_t stream) {
    const dim3 g(grid), b(128 * WN);
    if (tile) hipLaunchKernelGGL((medium_kernel<WN, MAXB, true, GROUPED, SWIGLU>), g, b, 0, stream, p);
    else hipLaunchKernelGGL((medium_kernel<WN, MAXB, false, GROUPED, SWIGLU>), g, b, 0, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_medium(const MediumParams& p, int grid, MediumConfig cfg, bool tile, bool swiglu, hipStream_t stream) {
    switch (cfg) {
        case MediumConfig::kWide: return launch_c<4, false, 4>(p, grid, tile, stream);
        case MediumConfig::kNarrow: return launch_c<2, false, 2>(p, grid, tile, stream);
        case MediumConfig::kGroupWide:
            return swiglu ? launch_c<4, true, 3, true>(p, grid, tile, stream) : launch_c<4, true, 3>(p, grid, tile, stream);
        case MediumConfig::kGroupNarrow:
            return swiglu ? launch_c<2, true, 2, true>(p, grid, tile, stream) : launch_c<2, true, 2>(p, grid, tile, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace tl
