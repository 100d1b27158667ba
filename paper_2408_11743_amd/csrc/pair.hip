// W4A16 GEMM for gfx950 with 64-row groups and two waves per SIMD:
// C[M,N] = A[M,K] * (s * (q - 8)), fp32 accumulation.
//
// The tiles, units and ranges are the stream kernel's with four 16-row blocks
// (64 rows x 128 columns per tile, gemm.hip).  Eight waves: four along N take 32
// columns each, and pairs of waves (w and w + 4) split K, one 128-row block each
// per stage; the pair's sums meet in LDS when a tile segment ends (Algorithm 1's
// reduction).  Codes are converted with the magic number (exact q - 8) and the
// group scale multiplies the fp16 weights (Section 3.4, "Dequantization and
// Tensor Cores", "Groups and Instruction Ordering").
//
// Everything a stage needs arrives by direct-to-LDS loads in a ring of three
// 50 KiB slots: two blocks' 64 activation rows (XOR-swizzled), each wave's words
// and scale row.  One barrier per stage, between a wave's second and third
// k-step: by then it holds the rest of the stage in registers, so the slot is
// free, and the next stage has landed.  The next stage's first rows, words and
// scales are read during the last two k-steps and its last rows during the
// first two, and the refill's loads are spread over those: with the loads in
// one burst per stage and two barriers around the operand reads the matrix cores
// idled at every stage.  Reads in flight never cross the loop's back edge or a
// branch: the compiler takes their registers as written and could move them.
//
// Bound: LDS bandwidth and vector issue (193 KiB of LDS traffic and 3.25 vector
// instructions per MFMA in a stage).  In one process with the kernel before it
// (a burst of loads and two barriers per stage): 8192 x 28672 at M = 64 44.2 us
// (45.7), per channel 39.4 (42.1), M = 33 39.4 (41.1); 4096 x 11008 at M = 128
// 21.3 (24.2), 1792 x 14592 at M = 114 12.9 (15.1).  Timing-only copies at
// M = 64: without the conversion 36.0, without the loads 36.6, without both 26.1.
#include <hip/hip_runtime.h>
#include <stdio.h>

#include "device.h"
#include "internal.h"

namespace marlin {
namespace {

using namespace dev;

constexpr int kPairP = 3;                      // ring slots
constexpr int kPairA = 64 * 256;               // a block's 64 rows x 128 k, bytes
constexpr int kPairWAt = 2 * kPairA;           // then the waves' words (2 KiB each)
constexpr int kPairSAt = kPairWAt + 8 * 2048;  // and scale rows (256 B each)
constexpr int kPairStage = kPairSAt + 8 * 256;
static_assert(kPairP * kPairStage <= 160 * 1024 - 64, "LDS");

template <bool PER_CHANNEL>
__global__ void __launch_bounds__(512, 1) w4a16_pair_kernel(GemmProblem p)
{
    constexpr int P = kPairP, kStage = kPairStage;
    constexpr int KS = 2;    // 128-row blocks of K per stage
    constexpr int MB = 4;    // 16-row blocks per wave
    constexpr int NB = 2;    // 16-column blocks per wave
    constexpr int kOwn = NB * MB / 2;  // blocks a wave keeps after the reduction
    constexpr int kDmaA = 4, kDmaW = 2, kDmaS = PER_CHANNEL ? 0 : 1;
    constexpr int kLoads = kDmaA + kDmaW + kDmaS;
    __shared__ __attribute__((aligned(16))) uint8_t ring[P * kStage];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wn = wave & 3, kg = wave >> 2;  // 32-column part, block of the stage
    const int lg = lane >> 4;
    const DequantConsts dq = dequant_consts();
    const int KU = p.KU;
    const int grid = gridDim.x;
    const int wg = xcd_local_wg(blockIdx.x, grid);
    const int u0 = range_start(p, wg, grid);
    const int u1 = range_start(p, wg + 1, grid);
    const int c_begin = tile_of(p, u0);
    const int c_end = tile_of(p, u1 - 1);  // the range's last tile
    const int k0 = u0 - c_begin * KU;
    const int k1 = u1 - c_end * KU;
    const int n_st = c_begin == c_end ? (k1 - k0 + KS - 1) / KS
                                      : (KU - k0 + KS - 1) / KS + (c_end - c_begin - 1) * ((KU + KS - 1) / KS) +
                                            (k1 + KS - 1) / KS;
    auto end_of = [&](int c) { return c == c_end ? k1 : c < c_end ? KU : 0; };

    // Tile c: column tile c / rg (128 columns), row group c % rg (64 rows).
    const uint32_t RG = (uint32_t)p.rg;
    auto col_of = [&](int c) -> uint32_t { return RG == 1 ? (uint32_t)c : (uint32_t)c / RG; };
    auto row0_of = [&](int c) -> int { return RG == 1 ? 0 : (int)((uint32_t)c - col_of(c) * RG) * 64; };
    auto rows_of = [&](int c) -> int {
        const int r = p.M - row0_of(c);
        return r < 64 ? r : 64;
    };
    // this wave's packed 64-column tile, and its half of it
    auto ptile_of = [&](int c) -> uint32_t { return col_of(c) * 2u + (uint32_t)(wn >> 1); };

    // ---- per-lane address parts ----
    // A: load i of this wave brings rows 4 wn + lg + 16 i of its block (all
    // with one swizzle)
    const uint32_t a_dma = (uint32_t)((4 * wn + lg) * p.K + (((lane & 15) ^ ((4 * wn + lg) & 15)) * 8)) * 2u;
    const uint32_t a_rows16 = (uint32_t)p.K * 32u;
    const uint32_t w_lane = (uint32_t)lane * 16u + (uint32_t)(wn & 1) * 2048u;
    const uint32_t s_lane = (uint32_t)(lane & 31) * 4u;
    const uint32_t w_bytes = (uint32_t)p.K * (uint32_t)(p.N / 2);
    const uint32_t s_bytes = (uint32_t)p.G * (uint32_t)p.N * 2u;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)ring;
    // Operand reads, k-step t: row l % 16 of a 16-row block, chunk (4t + l / 16)
    // ^ (l % 16).  A wave's row block mb is row block (mb + 2 kg) % 4 of the
    // tile, so that the blocks it keeps after the reduction are its first two.
    uint32_t a_rd[4][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const uint32_t at = lds0 + (uint32_t)(kg * kPairA + (lane & 15) * 256) +
                            (uint32_t)(((4 * t + lg) ^ (lane & 15)) << 4);
        a_rd[t][0] = at + (uint32_t)kg * 8192u;
        a_rd[t][1] = at + (uint32_t)(1 - kg) * 8192u;
    }
    const uint32_t w_rd = lds0 + (uint32_t)(kPairWAt + wave * 2048 + lane * 16);
    // this lane's column scale of block b: byte (cn / 4) * 32 + (nb * 4 + cn % 4) * 2, cn = lane % 16
    const uint32_t s_rd =
        lds0 + (uint32_t)(kPairSAt + wave * 256 + ((lane & 15) >> 2) * 32 + (wn & 1) * 16 + (lane & 3) * 2);

    // ---- load cursor ----
    int ld_c = c_begin, ld_ku = k0;
    int ld_end = end_of(ld_c);
    uint32_t ld_slot = 0;
    uint32_t ld_w, ld_s, a_bytes;
    const uint16_t *ld_a;
    auto ld_tile = [&]() {
        const int c = ld_end > 0 ? ld_c : c_end;
        ld_w = ptile_of(c) * (uint32_t)KU << 12;
        ld_s = ptile_of(c) * (uint32_t)p.G << 7;
        ld_a = p.A + (int64_t)row0_of(c) * p.K;
        a_bytes = (uint32_t)rows_of(c) * (uint32_t)p.K * 2u;
    };
    ld_tile();
    // Load i of a stage (0 .. kLoads - 1), all direct to LDS; a block past the
    // segment loads zeros through an empty descriptor.
    auto issue = [&](int i) {
        const int my = ld_ku + kg;
        const bool on = my < ld_end;
        uint32_t slot = lds0 + ld_slot;
        asm volatile("" : "+s"(slot));
        if (i < kDmaA) {
            const __amdgpu_buffer_rsrc_t ra =
                __builtin_amdgcn_make_buffer_rsrc((void *)ld_a, (short)0, on ? a_bytes : 0u, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                ra,
                (__attribute__((address_space(3))) void *)(uintptr_t)(slot + (uint32_t)(kg * kPairA + wn * 1024 + i * 4096)),
                16, (int)(a_dma + (uint32_t)i * a_rows16), my * 256, 0, 0);
        } else if (i < kDmaA + kDmaW) {
            const __amdgpu_buffer_rsrc_t rw =
                __builtin_amdgcn_make_buffer_rsrc((void *)p.W, (short)0, on ? w_bytes : 0u, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rw,
                (__attribute__((address_space(3))) void *)(uintptr_t)(
                    slot + (uint32_t)(kPairWAt + wave * 2048 + (i - kDmaA) * 1024)),
                16, (int)(w_lane + (uint32_t)(i - kDmaA) * 1024u), (int)(ld_w + ((uint32_t)my << 12)), 0,
                kAuxNonTemporal);
        } else if (i < kLoads) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc((void *)p.S, (short)0, on ? s_bytes : 0u, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void *)(uintptr_t)(slot + (uint32_t)(kPairSAt + wave * 256)), 4,
                (int)s_lane, (int)(ld_s + ((uint32_t)scale_row_of(my, p) << 7)), 0, 0);
        }
        issue_order_point();
    };
    auto advance_ld = [&]() {
        ld_slot = ld_slot == (uint32_t)((P - 1) * kStage) ? 0u : ld_slot + (uint32_t)kStage;
        ld_ku += KS;
        if (ld_ku >= ld_end) {
            ld_c += 1;
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

    u32x4_t av[4][MB];        // [k-step][row block]
    u32x4_t wv[NB], wn_[NB];  // packed words, k-step in the element: this stage's, the next one's
    uint32_t sv[NB];          // column scales as read
    half2_t s2[NB];
    half2_t nx[4];            // converted operand of the next four MFMAs
    uint32_t rd_slot = 0;
    auto read_a = [&](int t, int mb) {
        asm volatile("ds_read_b128 %0, %1 offset:%2"
                     : "=v"(av[t][mb])
                     : "v"(a_rd[t][mb >> 1] + rd_slot), "i"((mb & 1) * 4096));
    };
    auto read_w = [&](int b) {
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(wn_[b]) : "v"(w_rd + rd_slot), "i"(b * 1024));
    };
    auto read_s = [&](int b) {
        asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(sv[b]) : "v"(s_rd + rd_slot), "i"(b * 8));
    };
    auto landed_a = [&](int t) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(av[t][mb]));
    };
    auto landed_ws = [&]() {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            asm volatile("" : "+v"(wn_[b]));
            if constexpr (!PER_CHANNEL) {
                asm volatile("" : "+v"(sv[b]));
                s2[b] = as_h2(sv[b] | (sv[b] << 16));
            }
        }
    };
    // MFMA of k-step t, column block b and row block mb, with one quarter of
    // the next operand's conversion
    auto slot = [&](int t, int b, int mb, half8_t w, uint32_t next, half2_t ns) {
        acc[b][mb] = mfma(w, __builtin_bit_cast(half8_t, av[t][mb]), acc[b][mb]);
        nx[mb] = magic_quarter<!PER_CHANNEL>(next, mb, ns, dq);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto operand = [&]() {
        return half8_t{nx[0].x, nx[0].y, nx[1].x, nx[1].y, nx[2].x, nx[2].y, nx[3].x, nx[3].y};
    };

    // block j of this wave after the reduction = column block j / 2, row block 2 kg + j % 2
    auto own = [&](int j) { return wave * kOwn + j; };
    auto store_c = [&](int c, const float4_t *out) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));  // addresses formed here, not held across the loop
        const int lg = lane >> 4;
        const int r0 = row0_of(c) + kg * 32, rows = rows_of(c) - kg * 32;
        const uint32_t pt = ptile_of(c);
        half4_t cs[NB] = {};
        if constexpr (PER_CHANNEL) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
                cs[b] = *(const half4_t *)(p.S + (int64_t)pt * 64 + lg * 16 + ((wn & 1) * 2 + b) * 4);
        }
        auto rounded = [&](int b, int mb) -> half4_t {
            float4_t v = out[b * 2 + mb];
            if constexpr (PER_CHANNEL) {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] *= (float)cs[b][i];
            }
            return half4_t{(_Float16)v[0], (_Float16)v[1], (_Float16)v[2], (_Float16)v[3]};
        };
        uint16_t *const at = p.C + (int64_t)(pt * 64 + (wn & 1) * 32 + (lg & 1) * 16 + (lg >> 1) * 8);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const int m = mb * 16 + (lane & 15);
            const u32x4_t h = join_blocks(rounded(0, mb), rounded(1, mb));
            if (m < rows) *(u32x4_t *)(at + (int64_t)(r0 + m) * p.N) = h;
        }
    };
    constexpr int kSlotFloats = 8 * kOwn * 256;
    float *const my_slots = p.partials + (int64_t)wg * 2 * kSlotFloats;
    bool reduce_first = false;  // this wave sums the range's first tile at the end
    int cp_c = c_begin, cp_ku = k0, cp_begin = k0;
    int cp_end = end_of(cp_c);
    // Sum the two blocks' tiles: wave (wn, kg) keeps row blocks 2 kg and 2 kg + 1
    // and gives the others to its partner, through ring slot `at` (free: every
    // wave holds its stage's operands in registers, and the slot's refill is
    // issued after this).
    auto reduce_halves = [&](uint32_t at) {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        float4_t *const mine = reinterpret_cast<float4_t *>(ring + at + (uint32_t)wave * 4096u);
        const float4_t *const theirs = reinterpret_cast<const float4_t *>(ring + at + (uint32_t)(wave ^ 4) * 4096u);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) mine[(b * 2 + mb) * 64 + lane] = acc[b][2 + mb];
        lds_barrier();
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < 2; ++mb) acc[b][mb] += theirs[(b * 2 + mb) * 64 + lane];
        lds_barrier();
    };
    // A segment other than the range's last is complete: write C (whole tile),
    // or slot 0 (shared first tile) and arrive there.
    auto finish_segment = [&](uint32_t at) {
        reduce_halves(at);
        float4_t out[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) out[j] = acc[j / 2][j % 2];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[b][mb] = zero4;
        if (cp_begin != 0 || cp_end != KU) {
            int l = lane;
            asm volatile("" : "+v"(l));
#pragma unroll
            for (int j = 0; j < kOwn; ++j) store_partial16(my_slots, own(j), l, out[j]);
            wait_vmcnt<0>();
            reduce_first = arrive_by_wave(p, cp_c, wave, grid, l);
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
        for (int mb = 0; mb < MB; ++mb) read_a(t, mb);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        read_w(b);
        if constexpr (!PER_CHANNEL) read_s(b);
    }
    wait_lgkmcnt0();
#pragma unroll
    for (int t = 0; t < 4; ++t) landed_a(t);
    landed_ws();
#pragma unroll
    for (int b = 0; b < NB; ++b) wv[b] = wn_[b];
#pragma unroll
    for (int q = 0; q < 4; ++q) nx[q] = magic_quarter<!PER_CHANNEL>(wv[0][0], q, s2[0], dq);
    // k-steps 0 and 1 of stage 0
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const half8_t w = operand();
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) slot(t, b, mb, w, b == 0 ? wv[1][t] : wv[0][t + 1], s2[1 - b]);
        }

    for (int st = 0; st + 1 < n_st; ++st) {
        // Stage st + 1 has landed (P - 2 stages were issued after it), and
        // every wave holds the rest of stage st in registers.
        wait_vmcnt<(P - 2) * kLoads>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        const uint32_t old_slot = rd_slot;
        rd_slot = rd_slot == (uint32_t)((P - 1) * kStage) ? 0u : rd_slot + (uint32_t)kStage;
        // k-steps 2 and 3 of stage st; reads stage st + 1's words, scales and first rows
        constexpr int kFirst = PER_CHANNEL ? NB : 2 * NB;  // reads before the rows
#pragma unroll
        for (int t = 2; t < 4; ++t)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const half8_t w = operand();
                if (t == 3 && b == 1) {
                    wait_lgkmcnt_n(2 * MB);  // the words and scales: the rows' reads come after them
                    landed_ws();
                }
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int k = ((t - 2) * NB + b) * MB + mb;
                    slot(t, b, mb, w, b == 0 ? wv[1][t] : t == 2 ? wv[0][3] : wn_[0][0], s2[1 - b]);
                    if (k < NB) read_w(k);
                    else if (k < kFirst) read_s(k - NB);
                    else if (k < kFirst + 2 * MB) read_a((k - kFirst) / MB, (k - kFirst) % MB);
                }
            }
        wait_lgkmcnt0();
        landed_a(0);
        landed_a(1);
#pragma unroll
        for (int b = 0; b < NB; ++b) wv[b] = wn_[b];
        // stage st was its segment's last?
        if (cp_ku + KS >= cp_end) {
            finish_segment(old_slot);
            cp_c += 1;
            cp_ku = 0;
            cp_begin = 0;
            cp_end = end_of(cp_c);
        } else {
            cp_ku += KS;
        }
        // k-steps 0 and 1 of stage st + 1; refills stage st's slot and reads the last rows
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const half8_t w = operand();
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) {
                    const int k = (t * NB + b) * MB + mb;
                    slot(t, b, mb, w, b == 0 ? wv[1][t] : wv[0][t + 1], s2[1 - b]);
                    if (k < 2 * MB) read_a(2 + k / MB, k % MB);
                    if ((k & 1) && k / 2 < kLoads) issue(k / 2);
                }
            }
        wait_lgkmcnt0();  // read in the first k-step
        landed_a(2);
        landed_a(3);
        advance_ld();
    }
    // k-steps 2 and 3 of the last stage
#pragma unroll
    for (int t = 2; t < 4; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const half8_t w = operand();
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) slot(t, b, mb, w, b == 0 ? wv[1][t] : wv[0][3], s2[1 - b]);
        }
    wait_vmcnt<0>();
    lds_barrier();
    reduce_halves(0);

    // The last segment: whole, or the range's last tile (shared), whose sums
    // this wave adds from its registers if it completes the tile.
    float4_t last_out[kOwn], out[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn; ++j) last_out[j] = acc[j / 2][j % 2];
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
}

}  // namespace

hipError_t launch_pair_gemm(const GemmConfig &cfg, const GemmProblem &p, hipStream_t stream)
{
    if (cfg.sparse || cfg.mb != 4 || cfg.nb != 8) return hipErrorInvalidValue;
    GemmProblem arg = p;
    void *args[] = {&arg};
    const void *fn = p.group_units == 0 ? (const void *)&w4a16_pair_kernel<true>
                                        : (const void *)&w4a16_pair_kernel<false>;
    return hipLaunchKernel(fn, dim3(cfg.grid), dim3(512), args, 0, stream);
}

void pair_kernel_name(bool per_channel, char *buf, size_t n)
{
    snprintf(buf, n, "w4a16_pair_kernel<%s>", per_channel ? "true" : "false");
}

}  // namespace marlin
