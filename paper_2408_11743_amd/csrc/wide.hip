// W4A16 GEMM for gfx950 at prefill batches: C[M,N] = A[M,K] * (s * (q - 8)),
// fp32 accumulation, group scales on the fp16 weights.
//
//  * A work-group of eight waves (two per SIMD) owns a tile of 128 rows x 256
//    columns.  Four waves along N take one packed 64-column tile each; the two
//    waves of a column take the halves of every 128-row block of K, so each
//    owns 128 x 64 outputs, every converted word feeds eight MFMAs, and the
//    tile stays as small as with four waves.  The halves are summed in LDS when
//    a tile is done.
//  * A stage (one 128-row block: activation rows, XOR-swizzled, packed words, a
//    scale row per packed tile) arrives by direct-to-LDS loads in a ring of
//    three 49 KiB slots.  One barrier per stage, between a wave's two k-steps:
//    by then it holds the stage's operands in registers, so the slot is free,
//    and the next stage has landed.  The first rows, words and scales of the
//    next stage are read during the second k-step, its second rows during the
//    first, and the refill's loads are spread over the first.
//  * Codes are converted by the paper's magic number (exact q - 8; Section 3.4
//    "Dequantization and Tensor Cores") and multiplied by the group scale in
//    fp16, rounded once ("Groups and Instruction Ordering"), a quarter word
//    after every other MFMA (1.6 vector instructions per MFMA); per-channel
//    scales multiply the final sums.
//  * Reads in flight never cross the loop's back edge or a branch: the compiler
//    takes their registers as written and could move them.
//  * Partition and combination: as tile8.hip.
//
// Bound: vector issue and power (the shader clock is below 2.1 GHz here).  On
// 28672 x 8192: 1486 us at M = 4096 and 375 at 1024, against 1735 and 427 for
// four waves with the weights in a register ring (one wave per SIMD, loads in
// one burst per stage) and 1460 for a library fp16 GEMM at 4096; 8192 x 10240
// at M = 300 62 us (90).
#include <hip/hip_runtime.h>
#include <stdio.h>

#include "device.h"
#include "internal.h"

namespace marlin {
namespace {

using namespace dev;

struct WideShape {
    static constexpr int NW = 8;
    static constexpr int WN = 4;                   // waves along N (one packed tile each); two along K
    static constexpr int TR = 128;                 // rows of A per tile
    static constexpr int TC = 256;                 // columns per tile
    static constexpr int MB = 8, NB = 4;           // 16-row and 16-column blocks per wave
    static constexpr int kABytes = TR * 256;       // a stage: TR rows x 128 k of A,
    static constexpr int kWBytes = TC * 64;        // TC columns x 128 k of codes,
    static constexpr int kSBytes = WN * 256;       // and a scale row per packed tile
    static constexpr int kStage = kABytes + kWBytes + kSBytes;
    static constexpr int kDmaA = TR / (4 * NW);    // 1 KiB direct-to-LDS loads per wave
    static constexpr int kDmaW = TC / (16 * NW);
    static constexpr int P = 3;
    static_assert(P * kStage <= 160 * 1024 - 64, "LDS");
};

template <int MB, int NB, int P, typename SCALES>
__global__ void __launch_bounds__(512, 1) w4a16_wide_kernel(GemmProblem p)
{
    using S = WideShape;
    constexpr bool PER_CHANNEL = SCALES::per_channel;
    static_assert(MB == S::MB && NB == S::NB && P == S::P, "128 x 64 outputs per wave, three stages");
    constexpr int TR = S::TR, NW = S::NW;
    constexpr int kDmaA = S::kDmaA, kDmaW = S::kDmaW, kDmaS = PER_CHANNEL ? 0 : 1;
    constexpr int kLoads = kDmaA + kDmaW + kDmaS;
    constexpr int kStage = S::kStage;
    constexpr int kOwn = NB * MB / 2;  // blocks a wave keeps after the reduction
    __shared__ __attribute__((aligned(16))) uint8_t ring[P * kStage];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave & 3, kg = wave >> 2;  // packed tile of the column group, half of the 128 k
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
    // the scale row of this wave's packed tile (its 128 bytes twice)
    const uint32_t s_pt = (uint32_t)wn;
    const uint32_t s_lane = (uint32_t)(lane & 31) * 4u;
    const uint32_t w_bytes = (uint32_t)p.K * (uint32_t)(p.N / 2);
    const uint32_t s_bytes = (uint32_t)p.G * (uint32_t)p.N * 2u;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring;
    // Operand reads, k-step 2 kg + t of the block: row l % 16 of a 16-row
    // block, chunk (4 (2 kg + t) + l / 16) ^ (l % 16).  A wave's row block mb
    // is row block (mb + 4 kg) % 8 of the tile, so that the blocks it keeps
    // after the reduction are its first four.
    uint32_t a_rd[2][2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint32_t at =
            lds0 + (uint32_t)((lane & 15) * 256) + (uint32_t)(((4 * (2 * kg + t) + lg) ^ (lane & 15)) << 4);
        a_rd[t][0] = at + (uint32_t)kg * 16384u;
        a_rd[t][1] = at + (uint32_t)(1 - kg) * 16384u;
    }
    const uint32_t w_rd = lds0 + (uint32_t)(S::kABytes + wn * 4096 + lane * 16 + kg * 8);
    // this lane's column scale of block nb: byte (cn / 4) * 32 + (nb * 4 + cn % 4) * 2 of the row, cn = lane % 16
    const uint32_t s_rd =
        lds0 + (uint32_t)(S::kABytes + S::kWBytes + wn * 256 + ((lane & 15) >> 2) * 32 + (lane & 3) * 2);

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
                    slot + (uint32_t)(S::kABytes + S::kWBytes + wn * 256)),
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

    float4_t acc[NB][MB];
    const float4_t zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[b][mb] = zero4;

    u32x4_t av[2][MB];                   // [k-step][row block]
    typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
    u32x2_t wv[NB];                      // packed words, k-step in the element
    uint32_t sv[NB];                     // column scales as read
    half2_t s2[NB];
    half2_t nx[4];                       // converted operand of the next eight MFMAs
    uint32_t rd_slot = 0;
    auto read_a = [&](int t, int mb) {
        asm volatile("ds_read_b128 %0, %1 offset:%2"
                     : "=v"(av[t][mb])
                     : "v"(a_rd[t][mb >> 2] + rd_slot), "i"((mb & 3) * 4096));
    };
    auto read_w = [&](int b) {
        asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(wv[b]) : "v"(w_rd + rd_slot), "i"(b * 1024));
    };
    auto read_s = [&](int b) {
        asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(sv[b]) : "v"(s_rd + rd_slot), "i"(b * 8));
    };
    auto landed_a = [&](int t) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(av[t][mb]));
    };
    auto landed_ws = [&](int words) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b < words) asm volatile("" : "+v"(wv[b]));
            if constexpr (!PER_CHANNEL) asm volatile("" : "+v"(sv[b]));
        }
    };
    auto scales = [&]() {
        if constexpr (!PER_CHANNEL) {
#pragma unroll
            for (int b = 0; b < NB; ++b) s2[b] = as_h2(sv[b] | (sv[b] << 16));
        }
    };
    // The MFMA of k-step t, column block b and row block mb; every other one
    // also converts a quarter of the next operand's word
    auto slot = [&](int t, int b, int mb, half8_t w, uint32_t next, half2_t ns) {
        acc[b][mb] = mfma(w, __builtin_bit_cast(half8_t, av[t][mb]), acc[b][mb]);
        if ((mb & 1) == 0) nx[mb >> 1] = magic_quarter<!PER_CHANNEL>(next, mb >> 1, ns, dq);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto operand = [&]() {
        return half8_t{nx[0].x, nx[0].y, nx[1].x, nx[1].y, nx[2].x, nx[2].y, nx[3].x, nx[3].y};
    };

    // block j of this wave after the reduction = column block j / 4, row block 4 kg + j % 4
    auto own = [&](int j) { return wave * kOwn + j; };
    auto store_c = [&](int c, const float4_t *out) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // addresses formed here, not held across the loop
        const int lg = lane >> 4;
        const int r0 = row0_of(c) + kg * 64, rows = rows_of(c) - kg * 64;
        const uint32_t pt = cg_of(c) * 4u + (uint32_t)wn;
        if (pt >= n_tiles) return;
        half4_t cs[NB] = {};
        if constexpr (PER_CHANNEL) {
#pragma unroll
            for (int b = 0; b < NB; ++b) cs[b] = *(const half4_t *)(p.S + (int64_t)pt * 64 + lg * 16 + b * 4);
        }
        auto rounded = [&](int b, int mb) -> half4_t {
            float4_t v = out[b * 4 + mb];
            if constexpr (PER_CHANNEL) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] *= (float)cs[b][i];
            }
            return half4_t{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
        };
        uint16_t *const at = p.C + (int64_t)(pt * 64 + (lg & 1) * 16 + (lg >> 1) * 8);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            const int m = mb * 16 + (lane & 15);
#pragma unroll
            for (int b = 0; b < NB; b += 2) {
                const u32x4_t h = join_blocks(rounded(b, mb), rounded(b + 1, mb));
                if (m < rows) *(u32x4_t *)(at + (int64_t)(r0 + m) * p.N + b * 16) = h;
            }
        }
    };
    constexpr int kSlotFloats = NW * kOwn * 256;
    float *const my_slots = p.partials + (int64_t)wg * 2 * kSlotFloats;
    bool reduce_first = false, reduce_last = false;  // this wave sums that tile at the end
    int cp_c = c_begin, cp_ku = k0, cp_begin = k0;
    int cp_end = end_of(cp_c);
    // Sum the two K halves' tiles: wave (wn, kg) keeps row blocks 4 kg ..
    // 4 kg + 3 and gives the others to its partner, through ring slot `at`
    // (free: every wave holds its stage's operands in registers, and the slot's
    // refill is issued after this), four rounds of 4 KiB per wave.
    auto reduce_halves = [&](uint32_t at) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        float4_t *const mine = reinterpret_cast<float4_t *>(ring + at + (uint32_t)wave * 4096u);
        const float4_t *const theirs = reinterpret_cast<const float4_t *>(ring + at + (uint32_t)(wave ^ 4) * 4096u);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) mine[mb * 64 + lane] = acc[b][4 + mb];
            lds_barrier();
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) acc[b][mb] += theirs[mb * 64 + lane];
            lds_barrier();
        }
    };
    // A segment other than the last is complete: write C (whole tile), or the
    // slot of the range's last (1) or first (0) tile, and arrive at the tile.
    auto finish_segment = [&](uint32_t at) {
        reduce_halves(at);
        float4_t out[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) out[j] = acc[j / 4][j % 4];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[b][mb] = zero4;
        if (cp_begin != 0 || cp_end != KU) {
            int l = lane;
            asm volatile("" : "+v"(l));
            float *const slot = my_slots + (cp_c == c_end ? kSlotFloats : 0);
#pragma unroll
            for (int j = 0; j < kOwn; ++j) store_partial16(slot, own(j), l, out[j]);
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
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) read_a(t, mb);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        read_w(b);
        if constexpr (!PER_CHANNEL) read_s(b);
    }
    wait_lgkmcnt0();
    landed_a(0);
    landed_a(1);
    landed_ws(NB);
    scales();
#pragma unroll
    for (int q = 0; q < 4; ++q) nx[q] = magic_quarter<!PER_CHANNEL>(wv[0][0], q, s2[0], dq);
    // first k-step of stage 0
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const half8_t w = operand();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            slot(0, b, mb, w, b + 1 < NB ? wv[b + 1][0] : wv[0][1], s2[(b + 1) % NB]);
    }

    for (int st = 0; st + 1 < n_st; ++st) {
        // Stage st + 1 has landed (P - 2 stages were issued after it), and
        // every wave holds the rest of stage st in registers.
        wait_vmcnt<(P - 2) * kLoads>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t old_slot = rd_slot;
        rd_slot = rd_slot == (uint32_t)((P - 1) * kStage) ? 0u : rd_slot + (uint32_t)kStage;
        // second k-step of stage st; reads stage st + 1's first rows, words and scales
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const half8_t w = operand();
            if (b == NB - 1) {
                wait_lgkmcnt_n(1);  // all but word 3
                landed_a(0);
                landed_ws(NB - 1);
                scales();
            }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                slot(1, b, mb, w, b + 1 < NB ? wv[b + 1][1] : wv[0][0], s2[(b + 1) % NB]);
                const int k = b * MB + mb;
                if (k < MB) read_a(0, k);
                else if (!PER_CHANNEL && k < MB + NB) read_s(k - MB);
                // word b' is free once its last quarter is converted, one block ahead of its MFMAs
                if (mb == 7 && b < 2) read_w(b);
                if (mb == 2 && b == 2) read_w(2);
                if (mb == 7 && b == 2) read_w(3);
            }
        }
        wait_lgkmcnt0();
        asm volatile("" : "+v"(wv[NB - 1]));
        // stage st was its segment's last?
        if (cp_ku + 1 >= cp_end) {
            finish_segment(old_slot);
            cp_c = next_tile(cp_c);
            cp_ku = 0;
            cp_begin = 0;
            cp_end = end_of(cp_c);
        } else {
            cp_ku += 1;
        }
        // first k-step of stage st + 1; refills stage st's slot and reads the second k-step's rows
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const half8_t w = operand();
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                slot(0, b, mb, w, b + 1 < NB ? wv[b + 1][0] : wv[0][1], s2[(b + 1) % NB]);
                const int k = b * MB + mb;
                if (k < MB) read_a(1, k);
                if (k % 4 == 1 && k / 4 < kLoads) issue(k / 4);
            }
        }
        wait_lgkmcnt0();  // read three column blocks ago
        landed_a(1);
        advance_ld();
    }
    // second k-step of the last stage
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const half8_t w = operand();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) slot(1, b, mb, w, wv[b + 1 < NB ? b + 1 : b][1], s2[b + 1 < NB ? b + 1 : b]);
    }
    wait_vmcnt<0>();
    lds_barrier();
    reduce_halves(0);

    float4_t last_out[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn; ++j) last_out[j] = acc[j / 4][j % 4];
    // The last segment: whole, or the range's last tile (shared), whose sums
    // this wave adds from its registers if it completes the tile.
    float4_t out[kOwn];
    if (cp_begin == 0 && cp_end == KU) {
        store_c(cp_c, last_out);
    } else {
#pragma unroll
        for (int j = 0; j < kOwn; ++j) store_partial16(my_slots + kSlotFloats, own(j), lane, last_out[j]);
        wait_vmcnt<0>();
        if (arrive_by_wave(p, cp_c, wave, grid, lane)) {
            reduce_by_wave<kOwn>(p, cp_c, grid, kSlotFloats, lane, own, wg, last_out, out);
            store_c(cp_c, out);
        }
    }
    if (reduce_first) {
        reduce_by_wave<kOwn>(p, c_begin, grid, kSlotFloats, lane, own, -1, last_out, out);
        store_c(c_begin, out);
    }
    if (reduce_last) {
        reduce_by_wave<kOwn>(p, c_end, grid, kSlotFloats, lane, own, -1, last_out, out);
        store_c(c_end, out);
    }
}

}  // namespace

hipError_t launch_wide_gemm(const GemmConfig &cfg, const GemmProblem &p, hipStream_t stream)
{
    if (cfg.mb != 8 || cfg.nb != 4) return hipErrorInvalidValue;
    GemmProblem arg = p;
    void *args[] = {&arg};
    const void *fn = (p.group_units == 0) ? (const void *)&w4a16_wide_kernel<8, 4, 3, EightWaves<true>>
                                          : (const void *)&w4a16_wide_kernel<8, 4, 3, EightWaves<false>>;
    return hipLaunchKernel(fn, dim3(cfg.grid), dim3(512), args, 0, stream);
}

void wide_kernel_name(bool per_channel, char *buf, size_t n)
{
    snprintf(buf, n, "w4a16_wide_kernel<8, 4, 3, EightWaves<%s>>", per_channel ? "true" : "false");
}

}  // namespace marlin
