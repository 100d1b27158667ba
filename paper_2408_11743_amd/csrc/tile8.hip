// W4A16 GEMM for gfx950 beyond 64 rows, two waves per SIMD, group scales in
// fp32: C[M,N] = A[M,K] * (s * (q - 8)), fp32 accumulation.
//
//  * A work-group of eight waves owns a tile of 128 rows x 256 columns (WN x WM
//    = 4 x 2 waves of 64 x 64 outputs) or 64 rows x 256 columns (8 x 1 waves of
//    64 x 32).  A column tile past N is computed on zeros and not stored, so any
//    N the packed layout allows runs here.
//  * Everything a stage (one 128-row block of K) needs arrives by direct-to-LDS
//    loads in a ring of three (50 KiB) or four (34 KiB) slots: the activation
//    rows, XOR-swizzled, the packed words, and a row of scales per wave.
//  * One barrier per stage, before the last column block: by then a wave holds
//    all the stage's operands in registers, so its slot is free, and the next
//    stage has landed.  The last column block's MFMAs cover the reads of the
//    next stage's operands, each issued when its registers fall free, and the
//    refill's loads are spread over the MFMAs after the barrier: issued in one
//    burst at the stage's start (as tile.hip does), the loads hold the waves
//    back while the matrix cores idle.
//  * Each MFMA is followed by a quarter of the next operand's conversion (the
//    paper's magic number, exact q - 8) and one multiply-add that folds the
//    previous column block's 128-row product, times its group scale, into the
//    fp32 sums (3.25 vector instructions per MFMA).
//  * Reads in flight never cross the loop's back edge or a branch: the compiler
//    takes their registers as written and could move them.
//  * Partition: device.h's ranges over shared tiles, then whole tiles (the
//    hybrid, plan.cpp); shared tiles are combined wave by wave.
//
// Bound: vector issue and power.  At 28672 x 8192, M = 1024 (one run): 415 us,
// without the fold 378, without the conversion 396, without the loads 373,
// without the LDS reads 411, MFMAs alone 293; the shader clock drops to 1.95
// GHz.  Against the kernels it takes over from: 8192 x 28672 at M = 128 71.4 us
// (tile.hip's eight waves 80.6), 28672 x 8192 70.2 (row groups of 32: 78.9),
// 8192 x 10240 at M = 128 31.5 (row groups of 64: 39.7), and where no
// 128-column tile fits N (row groups of 32): 8192 x 12096 at M = 1748 355 us
// (1134).
#include <hip/hip_runtime.h>
#include <stdio.h>

#include "device.h"
#include "internal.h"

namespace marlin {
namespace {

using namespace dev;

template <int WN, int WM, int MBW, int NBW>
struct Tile8Shape {
    static constexpr int NW = WN * WM;             // waves per work-group
    static constexpr int TR = 16 * MBW * WM;       // rows of A per tile
    static constexpr int TC = 16 * NBW * WN;       // columns per tile
    static constexpr int kABytes = TR * 256;       // a stage: TR rows x 128 k of A,
    static constexpr int kWBytes = TC * 64;        // TC columns x 128 k of codes,
    static constexpr int kSBytes = NW * 256;       // and a scale row per wave
    static constexpr int kStage = kABytes + kWBytes + kSBytes;
    static constexpr int kDmaA = TR / (4 * NW);    // 1 KiB direct-to-LDS loads per wave
    static constexpr int kDmaW = TC / (16 * NW);
    static constexpr int kByLds = (160 * 1024 - 64) / kStage;
    static constexpr int P = kByLds < 4 ? kByLds : 4;
    static_assert(NW == 8, "two waves per SIMD");
    static_assert(MBW == 4 && (NBW == 2 || NBW == 4), "64 rows, half or whole packed tiles per wave");
    static_assert(kDmaA >= 1 && kDmaW >= 1, "every wave loads rows and weights");
    static_assert(P >= 3, "ring too shallow");
};

template <int WN, int WM, int MBW, int NBW, int KS, typename SCALES>
__global__ void __launch_bounds__(64 * WN * WM, 1) w4a16_tile_kernel(GemmProblem p)
{
    static_assert(KS == 1, "one 128-row block of K per stage");
    constexpr bool PER_CHANNEL = SCALES::per_channel;
    using S = Tile8Shape<WN, WM, MBW, NBW>;
    constexpr int P = S::P, TR = S::TR, NW = S::NW;
    constexpr int kDmaA = S::kDmaA, kDmaW = S::kDmaW, kDmaS = PER_CHANNEL ? 0 : 1;
    constexpr int kLoads = kDmaA + kDmaW + kDmaS;
    constexpr int kStage = S::kStage;
    constexpr int kBlocks = NBW * MBW;
    constexpr int kGroups = 4 * MBW;  // MFMAs of one column block and stage
    constexpr int kSRd = PER_CHANNEL ? 0 : NBW / 2;  // scale reads per stage
    static_assert((P - 2) * kLoads < 64, "vmcnt range");
    __shared__ __attribute__((aligned(16))) uint8_t ring[P * kStage];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave % WN, wm = wave / WN;
    const int lg = lane >> 4;
    const DequantConsts dq = dequant_consts();
    const int KU = p.KU;
    const int grid = gridDim.x;
    const int wg = xcd_local_wg(blockIdx.x, grid);
    const int u0 = range_start(p, wg, grid);
    const int u1 = range_start(p, wg + 1, grid);
    // The work-group's stages: its range of the shared tiles (0 .. n_shared - 1),
    // if any, then whole tiles n_shared + wg, n_shared + wg + grid, ...
    const int n_shared = p.units / KU;
    const int c_end = u1 > u0 ? tile_of(p, u1 - 1) : -1;  // the range's last tile
    const int k1 = u1 - c_end * KU;
    const int c_begin = u1 > u0 ? tile_of(p, u0) : n_shared + wg;
    const int k0 = u1 > u0 ? u0 - c_begin * KU : 0;
    const int n_st = u1 - u0 + (p.tiles - n_shared) / grid * KU;
    // The tile after c (p.tiles or more: none), and the end of tile c's segment.
    auto next_tile = [&](int c) { return c < c_end ? c + 1 : c < n_shared ? n_shared + wg : c + grid; };
    auto end_of = [&](int c) { return c == c_end ? k1 : c < p.tiles ? KU : 0; };

    // Tile c: column group c / rg (TC columns), row group c % rg (TR rows).
    const uint32_t RG = (uint32_t)p.rg;
    auto cg_of = [&](int c) -> uint32_t { return RG == 1 ? (uint32_t)c : (uint32_t)c / RG; };
    auto row0_of = [&](int c) -> int { return RG == 1 ? 0 : (int)((uint32_t)c - cg_of(c) * RG) * TR; };
    auto rows_of = [&](int c) -> int {
        const int r = p.M - row0_of(c);
        return r < TR ? r : TR;
    };
    const uint32_t n_tiles = (uint32_t)p.N / 64u;  // packed 64-column tiles

    // ---- per-lane address parts ----
    // A: load i of this wave brings rows r0 + lg + 16 i (all with one swizzle,
    // so that one register and a scalar step address every load)
    const int r0_dma = (wave & 3) * 4 + (wave >> 2) * (kDmaA * 16);
    const uint32_t a_dma =
        (uint32_t)((r0_dma + lg) * p.K + (((lane & 15) ^ ((r0_dma + lg) & 15)) * 8)) * 2u;
    const uint32_t a_rows16 = (uint32_t)p.K * 32u;
    // this wave's weight loads: KiB kDmaW * wave .. of the stage's TC / 16 (four per packed tile)
    const uint32_t w_pt = (uint32_t)(kDmaW * wave) >> 2;
    const uint32_t w_lane = (uint32_t)lane * 16u + (((uint32_t)(kDmaW * wave) & 3u) << 10);
    // the scale row of the packed tile that holds this wave's columns (its 128 bytes twice)
    const uint32_t s_pt = (uint32_t)(wn * NBW) >> 2;
    const uint32_t s_lane = (uint32_t)(lane & 31) * 4u;
    const uint32_t w_bytes = (uint32_t)p.K * (uint32_t)(p.N / 2);
    const uint32_t s_bytes = (uint32_t)p.G * (uint32_t)p.N * 2u;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring;
    uint32_t a_rd[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
        a_rd[t] = lds0 + (uint32_t)((wm * 16 * MBW + (lane & 15)) * 256 + (((4 * t + lg) ^ (lane & 15)) << 4));
    const uint32_t w_rd = lds0 + (uint32_t)(S::kABytes + wn * NBW * 1024 + lane * 16);
    const uint32_t s_rd = lds0 + (uint32_t)(S::kABytes + S::kWBytes + wave * 256 + lg * 32 + (NBW == 2 ? (wn & 1) * 16 : 0));

    // ---- load cursor ----
    int ld_c = c_begin, ld_ku = k0;
    int ld_end = end_of(ld_c);
    uint32_t ld_slot = 0;  // byte offset of the ring slot
    uint32_t ld_w, ld_wbytes, ld_s, ld_sbytes, a_bytes;
    const uint16_t *ld_a;
    auto ld_tile = [&]() {
        const uint32_t pt0 = cg_of(ld_c) * (uint32_t)(S::TC / 64);
        const bool in = ld_end > 0;
        ld_w = (pt0 + w_pt) * (uint32_t)KU << 12;
        ld_wbytes = in && pt0 + w_pt < n_tiles ? w_bytes : 0u;
        ld_s = (pt0 + s_pt) * (uint32_t)p.G << 7;
        ld_sbytes = in && pt0 + s_pt < n_tiles ? s_bytes : 0u;
        const int c = in ? ld_c : 0;
        ld_a = p.A + (int64_t)row0_of(c) * p.K;
        a_bytes = in ? (uint32_t)rows_of(c) * (uint32_t)p.K * 2u : 0u;
    };
    ld_tile();
    // Load i of a stage (0 .. kLoads - 1), all direct to LDS.
    auto issue = [&](int i) {
        uint32_t slot = lds0 + ld_slot;
        asm volatile("" : "+s"(slot));
        if (i < kDmaA) {
            const __amdgpu_buffer_rsrc_t ra =
                __builtin_amdgcn_make_buffer_rsrc((void *)ld_a, (short)0, a_bytes, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                ra,
                (__attribute__((address_space(3))) void *)(uintptr_t)(slot + (uint32_t)(r0_dma * 256 + i * 4096)),
                16, (int)(a_dma + (uint32_t)i * a_rows16), ld_ku * 256, 0, 0);
        } else if (i < kDmaA + kDmaW) {
            const __amdgpu_buffer_rsrc_t rw =
                __builtin_amdgcn_make_buffer_rsrc((void *)p.W, (short)0, ld_wbytes, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rw,
                (__attribute__((address_space(3))) void *)(uintptr_t)(
                    slot + (uint32_t)(S::kABytes + (wave * kDmaW + i - kDmaA) * 1024)),
                16, (int)(w_lane + (uint32_t)(i - kDmaA) * 1024u), (int)(ld_w + ((uint32_t)ld_ku << 12)), 0,
                kAuxNonTemporal);
        } else if (i < kLoads) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc((void *)p.S, (short)0, ld_sbytes, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs,
                (__attribute__((address_space(3))) void *)(uintptr_t)(
                    slot + (uint32_t)(S::kABytes + S::kWBytes + wave * 256)),
                4, (int)s_lane, (int)(ld_s + ((uint32_t)scale_row_of(ld_ku, p) << 7)), 0, 0);
        }
        issue_order_point();
    };
    auto advance_ld = [&]() {
        ld_slot = ld_slot == (uint32_t)((P - 1) * kStage) ? 0u : ld_slot + (uint32_t)kStage;
        if (++ld_ku >= ld_end) {
            ld_c = next_tile(ld_c);
            ld_ku = 0;
            ld_end = end_of(ld_c);
            ld_tile();
        }
    };

#pragma unroll
    for (int j = 0; j < P; ++j) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) issue(i);
        advance_ld();
    }

    float4_t acc[NBW][MBW], tmp[2][MBW];
    const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NBW; ++b)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) acc[b][mb] = zero4;

    // ---- operands of one stage, all in registers ----
    u32x4_t av[4][MBW];   // [k-step][row block]
    u32x4_t wv[NBW];      // packed words, k-step in the element
    u32x4_t sv[2];        // this lane's scales: halves 4b .. 4b + 3 for column block b
    u32x4_t s_prev;       // element 0, 1: the last column block's of the stage before
    half2_t nx[4];        // converted operand of the next four MFMAs
    uint32_t rd_slot = 0;

    auto read_a = [&](int t, int mb) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(av[t][mb]) : "v"(a_rd[t] + rd_slot), "i"(mb * 4096));
    };
    auto read_w = [&](int b) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(wv[b]) : "v"(w_rd + rd_slot), "i"(b * 1024));
    };
    auto read_s = [&](int i) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(sv[i]) : "v"(s_rd + rd_slot), "i"(i * 16));
    };
    auto landed_a = [&](int t) {
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) asm volatile("" : "+v"(av[t][mb]));
    };
    auto scale_of = [&](int b, int i) -> float {  // this stage's
        const half8_t h = __builtin_bit_cast(half8_t, sv[b >> 1]);
        return (float)h[(b & 1) * 4 + i];
    };
    // fold element (mb, i) of column block b's product (in tmp[b & 1])
    auto fold = [&](int b, int mb, int i, bool prev) {
        float v;
        if constexpr (PER_CHANNEL) {
            v = acc[b][mb][i] + tmp[b & 1][mb][i];
        } else {
            const half8_t hp = __builtin_bit_cast(half8_t, s_prev);
            v = __builtin_fmaf(tmp[b & 1][mb][i], prev ? (float)hp[i] : scale_of(b, i), acc[b][mb][i]);
        }
        asm volatile("" : "+v"(v));  // here, not sunk to the next use
        acc[b][mb][i] = v;
    };

    // MFMA k of column block b (k-step k / MBW, row block k % MBW), and with
    // it one quarter of the next operand's conversion and one folded value
    // of column block fb (-1: none).  `next`: the word converted
    auto slot = [&](int b, int k, half8_t w, uint32_t next, int fb, bool prev) {
        const int t = k / MBW, mb = k % MBW;
        tmp[b & 1][mb] = mfma(w, __builtin_bit_cast(half8_t, av[t][mb]), t == 0 ? zero4 : tmp[b & 1][mb]);
        nx[mb] = magic_quarter<false>(next, mb, half2_t{}, dq);
        if (fb >= 0) fold(fb, mb, t, prev);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto operand = [&]() {
        return half8_t{nx[0].x, nx[0].y, nx[1].x, nx[1].y, nx[2].x, nx[2].y, nx[3].x, nx[3].y};
    };

    // block j of this wave = column block j / MBW, row block j % MBW; slot index wave*kBlocks + j
    auto own = [&](int j) { return wave * kBlocks + j; };
    auto store_c = [&](int c, const float4_t *out) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // addresses formed here, not held across the loop
        const int lg = lane >> 4;
        const int r0 = row0_of(c) + wm * 16 * MBW, rows = rows_of(c) - wm * 16 * MBW;
        const uint32_t nb0 = (cg_of(c) * WN + (uint32_t)wn) * NBW;  // first 16-column block
        if ((nb0 >> 2) >= n_tiles) return;
        half4_t cs[NBW] = {};
        if constexpr (PER_CHANNEL) {
#pragma unroll
            for (int b = 0; b < NBW; ++b)
                cs[b] = *(const half4_t *)(p.S + (int64_t)((nb0 + b) >> 2) * 64 + lg * 16 + ((nb0 + b) & 3u) * 4);
        }
        auto rounded = [&](int b, int mb) -> half4_t {
            float4_t v = out[b * MBW + mb];
            if constexpr (PER_CHANNEL) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] *= (float)cs[b][i];
            }
            return half4_t{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
        };
        uint16_t *const at = p.C + (int64_t)(nb0 * 16 + (lg & 1) * 16 + (lg >> 1) * 8);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) {
            const int m = mb * 16 + (lane & 15);
#pragma unroll
            for (int b = 0; b < NBW; b += 2) {
                const u32x4_t h = join_blocks(rounded(b, mb), rounded(b + 1, mb));
                if (m < rows) *(u32x4_t *)(at + (int64_t)(r0 + m) * p.N + b * 16) = h;
            }
        }
    };
    constexpr int kSlotFloats = NW * kBlocks * 256;
    float *const my_slots = p.partials + (int64_t)wg * 2 * kSlotFloats;
    bool reduce_first = false, reduce_last = false;  // this wave sums that tile at the end
    int cp_c = c_begin, cp_ku = k0, cp_begin = k0;
    int cp_end = end_of(cp_c);
    // A segment other than the last is complete: write C (whole tile), or the
    // slot of the range's last (1) or first (0) tile, and arrive at the tile.
    auto finish_segment = [&]() {
        float4_t out[kBlocks];
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            out[j] = acc[j / MBW][j % MBW];
            acc[j / MBW][j % MBW] = zero4;
        }
        if (cp_begin != 0 || cp_end != KU) {
            int l = lane;
            asm volatile("" : "+v"(l));
            float *const slot = my_slots + (cp_c == c_end ? kSlotFloats : 0);
#pragma unroll
            for (int j = 0; j < kBlocks; ++j) store_partial16(slot, own(j), l, out[j]);
            wait_vmcnt<0>();
            const bool last = arrive_by_wave(p, cp_c, wave, grid, l);
            if (cp_c == c_end)
                reduce_last = last;
            else
                reduce_first = last;
        } else {
            store_c(cp_c, out);
        }
    };

    // Stage 0's operands.
    wait_vmcnt<(P - 1) * kLoads>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) read_a(t, mb);
#pragma unroll
    for (int b = 0; b < NBW; ++b) read_w(b);
#pragma unroll
    for (int i = 0; i < kSRd; ++i) read_s(i);
    s_prev = u32x4_t{0u, 0u, 0u, 0u};
    wait_lgkmcnt0();
#pragma unroll
    for (int t = 0; t < 4; ++t) landed_a(t);
#pragma unroll
    for (int b = 0; b < NBW; ++b) asm volatile("" : "+v"(wv[b]));
#pragma unroll
    for (int i = 0; i < kSRd; ++i) asm volatile("" : "+v"(sv[i]));
#pragma unroll
    for (int q = 0; q < 4; ++q) nx[q] = magic_quarter<false>(wv[0][0], q, half2_t{}, dq);
    // column blocks 0 .. NBW - 2 of a stage
    auto mid_blocks = [&](int b_from) {
#pragma unroll
        for (int b = b_from; b < NBW - 1; ++b) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const half8_t w = operand();
                const uint32_t next = t < 3 ? wv[b][t + 1] : wv[b + 1][0];
#pragma unroll
                for (int mb = 0; mb < MBW; ++mb) slot(b, t * MBW + mb, w, next, b - 1, false);
            }
        }
    };
    mid_blocks(0);

    constexpr int L = NBW - 1;  // last column block
    for (int st = 0; st + 1 < n_st; ++st) {
        // Stage st + 1 has landed (loads issued after it: P - 2 stages), and
        // every wave holds stage st's operands in registers: its slot is free.
        wait_vmcnt<(P - 2) * kLoads>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        rd_slot = rd_slot == (uint32_t)((P - 1) * kStage) ? 0u : rd_slot + (uint32_t)kStage;
        // last column block of stage st; its operands' registers take stage st + 1's as they fall free
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const half8_t w = operand();
            if (t == 3) {
                // next stage's first word: read at the first slots
                wait_lgkmcnt_n(8 + NBW - 2);  // after wv[0]: NBW - 2 words, 2 k-steps of rows
                asm volatile("" : "+v"(wv[0]));
            }
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb) {
                const int k = t * MBW + mb;
                slot(L, k, w, t < 3 ? wv[L][t + 1] : wv[0][0], L - 1, false);
                if (k < NBW - 1) read_w(k);
                if (k >= MBW) read_a(k / MBW - 1, mb);
                if (k % 3 == 0 && k / 3 < kLoads) issue(k / 3);
            }
        }
        read_w(L);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) read_a(3, mb);
        if constexpr (!PER_CHANNEL) {
            s_prev[0] = sv[L >> 1][(L & 1) * 2];
            s_prev[1] = sv[L >> 1][(L & 1) * 2 + 1];
        }
        // column block 0 of stage st + 1; folds the last one of stage st
        constexpr int kTail = 1 + MBW;  // reads after k-step 2's rows
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const half8_t w = operand();
            if (t == 0) wait_lgkmcnt_n(kTail + 2 * MBW);
            if (t == 1) wait_lgkmcnt_n(kTail + MBW + kSRd);
            if (t == 2) wait_lgkmcnt_n(kTail + kSRd);
            if (t == 3) wait_lgkmcnt0();
            landed_a(t);
            const uint32_t next = t < 3 ? wv[0][t + 1] : wv[1 % NBW][0];
            if (t == 3) {
#pragma unroll
                for (int b = 1; b < NBW; ++b) asm volatile("" : "+v"(wv[b]));
#pragma unroll
                for (int i = 0; i < kSRd; ++i) asm volatile("" : "+v"(sv[i]));
            }
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb) {
                const int k = t * MBW + mb;
                slot(0, k, w, t < 3 ? next : wv[1][0], L, true);
                if (k < kSRd) read_s(k);
                if (16 / 3 + 1 + k / 3 < kLoads && k % 3 == 0) issue(16 / 3 + 1 + k / 3);
            }
        }
        advance_ld();
        // stage st was its segment's last?
        if (cp_ku + 1 >= cp_end) {
            finish_segment();
            cp_c = next_tile(cp_c);
            cp_ku = 0;
            cp_begin = 0;
            cp_end = end_of(cp_c);
        } else {
            cp_ku += 1;
        }
        mid_blocks(1);
    }
    // last column block of the last stage
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const half8_t w = operand();
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb) slot(L, t * MBW + mb, w, wv[L][t < 3 ? t + 1 : 3], L - 1, false);
    }
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) fold(L, mb, i, false);
    wait_vmcnt<0>();

    float4_t last_out[kBlocks];
#pragma unroll
    for (int j = 0; j < kBlocks; ++j) last_out[j] = acc[j / MBW][j % MBW];
    // The last segment: whole, or the range's last tile (shared), whose sums
    // this wave adds from its registers if it completes the tile.
    float4_t out[kBlocks];
    if (cp_begin == 0 && cp_end == KU) {
        store_c(cp_c, last_out);
    } else {
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) store_partial16(my_slots + kSlotFloats, own(j), lane, last_out[j]);
        wait_vmcnt<0>();
        if (arrive_by_wave(p, cp_c, wave, grid, lane)) {
            reduce_by_wave<kBlocks>(p, cp_c, grid, kSlotFloats, lane, own, wg, last_out, out);
            store_c(cp_c, out);
        }
    }
    if (reduce_first) {
        reduce_by_wave<kBlocks>(p, c_begin, grid, kSlotFloats, lane, own, -1, last_out, out);
        store_c(c_begin, out);
    }
    if (reduce_last) {
        reduce_by_wave<kBlocks>(p, c_end, grid, kSlotFloats, lane, own, -1, last_out, out);
        store_c(c_end, out);
    }
}

}  // namespace

template <int WN, int WM, int NBW>
static hipError_t launch_tile8(const GemmConfig &cfg, const GemmProblem &p, hipStream_t stream)
{
    GemmProblem arg = p;
    void *args[] = {&arg};
    const void *fn = (p.group_units == 0) ? (const void *)&w4a16_tile_kernel<WN, WM, 4, NBW, 1, EightWaves<true>>
                                          : (const void *)&w4a16_tile_kernel<WN, WM, 4, NBW, 1, EightWaves<false>>;
    return hipLaunchKernel(fn, dim3(cfg.grid), dim3(512), args, 0, stream);
}

hipError_t launch_tile8_gemm(const GemmConfig &cfg, const GemmProblem &p, hipStream_t stream)
{
    switch (cfg.tile_wm * 10 + cfg.nb) {
    case 24: return launch_tile8<4, 2, 4>(cfg, p, stream);
    case 12: return launch_tile8<8, 1, 2>(cfg, p, stream);
    default: return hipErrorInvalidValue;
    }
}

void tile8_kernel_name(const GemmConfig &cfg, bool per_channel, char *buf, size_t n)
{
    snprintf(buf, n, "w4a16_tile_kernel<%d, %d, 4, %d, 1, EightWaves<%s>>", 8 / cfg.tile_wm, cfg.tile_wm, cfg.nb,
             per_channel ? "true" : "false");
}

}  // namespace marlin
