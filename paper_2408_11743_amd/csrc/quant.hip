// Weight quantiser for gfx950: fp16 W[K][N] -> 4-bit codes q[K][N] and fp16
// scales s[K/g][N] in the format the GEMM consumes, w = s * (q - 8).
//
// Uniform quantisation (Section 2.2, Eq. 1) in its symmetric form: a group of
// g consecutive weights of a column is mapped onto the range [-a, a] with 15
// steps of s = 2a / 15 and the fixed zero point 8, q = clamp(rint(v * (1/s))
// + 8, 0, 15).  The clipping threshold a = r * max|v| is searched per group over
// the caller's ratios r, keeping the one with the smallest reconstruction
// error sum (v - s(q - 8))^2 (Section 2.2; the group-wise clipping search of
// Section 3.5).  GPTQ's error feedback needs calibration data and is not
// part of this quantiser.
//
// Every decision (the rounding of each code, the choice of the ratio) is an
// fp32 computation in a fixed order: the stored fp16 scale is formed first,
// codes use its fp32 reciprocal, each thread sums its group sequentially,
// and no multiply-add is contracted, so the result is the same bits on any
// device and in any launch shape.
//
// With g = 128 one thread owns one (group, column) and holds its values in
// registers for the whole search; other groups are searched with a lane per
// (column, ratio) over LDS copies of 128-row chunks.  W comes row-major, [K][N],
// and leaves as codes and scales, or as a linear layer's [N][K] and leaves
// packed (the GEMM's layout, pack.hip), so that a layer's load is one kernel.
//
// Bound: vector issue.  Per weight and ratio the search needs a product, a
// rounding, a clamp, the difference, its square and the sum; the difference
// v - t s is one fused multiply-add, which rounds as the two operations do
// because t s (4 by 11 bits) is exact.  28672 x 8192 with ten ratios: 332 us at
// g = 128 (seven operations per term: 393; 21 clocks per term and SIMD, of which
// the rounding and the clamp, at half rate, take 9); 4096 x 11008 per channel
// 230 us (a thread per group re-reading it for each ratio: 3650).  Loading a
// 4096 x 11008 linear layer: 83 us (transposed copy, quantiser and packer: 427).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.h"
#include "quant.h"

namespace marlin {
namespace {

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct QuantArgs {
    const uint16_t *W;
    uint8_t *q;   // codes [K][N], or packed words
    uint16_t *s;  // scales [G][N], or packed scales
    int K, N, g;
    int n_ratios;
    float ratios[kMaxQuantRatios];
};

__device__ __forceinline__ float h2f(uint16_t bits) { return (float)__builtin_bit_cast(_Float16, bits); }

// Code offset t = q - 8 of v for the reciprocal inv of a non-zero scale.
__device__ __forceinline__ float code_of(float v, float inv)
{
    float t = __builtin_rintf(v * inv);
    return __builtin_fminf(__builtin_fmaxf(t, -8.0f), 7.0f);
}

// Scale of the clipping threshold r * max|v|.
__device__ __forceinline__ _Float16 scale_of(float ratio, float amax)
{
#pragma clang fp contract(off)
    const float lim = ratio * amax;
    return (_Float16)((lim + lim) / 15.0f);
}

// One term of the reconstruction error: (v - s t)^2, the product s t exact.
__device__ __forceinline__ float error_term(float err, float v, float inv, float sf)
{
#pragma clang fp contract(off)
    const float d = __builtin_fmaf(-code_of(v, inv), sf, v);
    return err + d * d;
}

// Eight codes (offsets t of rows j = 0..7, times `on`, 0 for a zero scale) -> one
// packed word, code j in nibble (j >> 1) + 4 (j & 1).  Halves of four nibbles
// are exact fp32 sums.
template <typename F>
__device__ __forceinline__ uint32_t pack_word(F t, float on)
{
    const float bias = 8.0f * 4369.0f;  // 8 in four nibbles
    float lo = bias, hi = bias;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        lo = __builtin_fmaf(t(2 * i), (float)(1 << (4 * i)) * on, lo);
        hi = __builtin_fmaf(t(2 * i + 1), (float)(1 << (4 * i)) * on, hi);
    }
    return (uint32_t)lo | ((uint32_t)hi << 16);
}

// Index of scale row r, column n in the packed scales.
__device__ __forceinline__ int64_t packed_scale_index(int r, int n, int G)
{
    return ((((int64_t)(n >> 6) * G + r) * 4 + ((n >> 2) & 3)) * 4 + ((n >> 4) & 3)) * 4 + (n & 3);
}

// g = 128: one thread per (group, column).  LINEAR: W is [N][K] (a thread reads
// its 256 bytes by 16-byte loads) and the results are packed; else W is [K][N]
// (every row of a group is one coalesced 2-byte-per-lane load).  The values
// stay in registers (two waves per SIMD), indexed by constants only.
template <bool LINEAR>
__global__ void __launch_bounds__(256) quantize128_kernel(QuantArgs a)
{
#pragma clang fp contract(off)
    constexpr int g = 128;
    const int n = blockIdx.x * 256 + (int)threadIdx.x;
    if (n >= a.N) return;
    const int gr = blockIdx.y;
    float v[g];
    if constexpr (LINEAR) {
        const half8_t *row = (const half8_t *)(a.W + (int64_t)n * a.K + (int64_t)gr * g);
#pragma unroll
        for (int i = 0; i < g / 8; ++i) {
            const half8_t h = row[i];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[8 * i + j] = (float)h[j];
        }
    } else {
        const uint16_t *col = a.W + (int64_t)gr * g * a.N + n;
#pragma unroll
        for (int k = 0; k < g; ++k) v[k] = h2f(col[(int64_t)k * a.N]);
    }
    // kept as fp32: reading fp16 halves in place halves the rate of an operation
#pragma unroll
    for (int k = 0; k < g; ++k) asm volatile("" : "+v"(v[k]));
    float amax = 0.0f;
#pragma unroll
    for (int k = 0; k < g; ++k) amax = __builtin_fmaxf(amax, __builtin_fabsf(v[k]));

    float best_err = __builtin_inff();
    _Float16 best = (_Float16)0.0f;
    for (int i = 0; i < a.n_ratios; ++i) {
        const _Float16 s16 = scale_of(a.ratios[i], amax);
        float sf = (float)s16;
        asm volatile("" : "+v"(sf));
        // a zero scale codes everything as 8: inv = 0 gives t = 0, the group's energy
        const float inv = sf == 0.0f ? 0.0f : 1.0f / sf;
        float err = 0.0f;
#pragma unroll
        for (int k = 0; k < g; ++k) err = error_term(err, v[k], inv, sf);
        if (err < best_err) {
            best_err = err;
            best = s16;
        }
    }

    const float sf = (float)best;
    const float inv = sf == 0.0f ? 0.0f : 1.0f / sf, on = sf == 0.0f ? 0.0f : 1.0f;
    if constexpr (LINEAR) {
        uint32_t *w = (uint32_t *)a.q + (((int64_t)(n >> 6) * (a.K / 128) + gr) * 4 + ((n >> 4) & 3)) * 256 + (n & 15) * 4;
#pragma unroll
        for (int lg = 0; lg < 4; ++lg) {
            u32x4_t word;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                word[t] = pack_word([&](int j) { return code_of(v[32 * t + 8 * lg + j], inv); }, on);
            *(u32x4_t *)(w + lg * 64) = word;
        }
        a.s[packed_scale_index(gr, n, a.K / g)] = __builtin_bit_cast(uint16_t, best);
    } else {
        uint8_t *qc = a.q + (int64_t)gr * g * a.N + n;
#pragma unroll
        for (int k = 0; k < g; ++k) qc[(int64_t)k * a.N] = (uint8_t)(int)__builtin_fmaf(code_of(v[k], inv), on, 8.0f);
        a.s[(int64_t)gr * a.N + n] = __builtin_bit_cast(uint16_t, best);
    }
}

// Other groups (multiples of 128 rows, up to a whole column): a block owns 16
// columns of one group and a lane one of them and one ratio (four ratios per
// wave), so a group's ratios are searched in parallel: a thread per group alone
// leaves the chip idle (a per-channel layer has N groups) behind a chain of K
// sums per ratio.  The block's waves bring 128-row chunks to LDS in turn
// (double-buffered; 16-byte reads, four lanes of one column read together),
// first for max|v|, then for the search, and code the chunks in parallel.
constexpr int kCols = 16;
constexpr int kPitch = 128 + 8;  // halves per column and chunk: 16-byte reads of 16 columns hit all banks

template <bool LINEAR>
__global__ void __launch_bounds__(1024) quantize_group_kernel(QuantArgs a)
{
#pragma clang fp contract(off)
    __shared__ __attribute__((aligned(16))) uint16_t chunk[2][kCols * kPitch];
    __shared__ float shared_max[16][kCols];
    __shared__ float errs[kMaxQuantRatios][kCols];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int c = lane & 15;           // column of the block
    const int blk = dev::xcd_local_wg(blockIdx.x, gridDim.x);  // neighbours share the lines of a row in one L2
    const int n0 = blk % (a.N / kCols) * kCols, gr = blk / (a.N / kCols);
    const int chunks = a.g / 128;
    const int64_t k0 = (int64_t)gr * a.g;

    // Eight values (rows 8 o .. 8 o + 7 of chunk ch) of column cc.
    auto load8 = [&](int ch, int o, int cc) -> half8_t {
        const int64_t k = k0 + ch * 128 + 8 * o;
        if constexpr (LINEAR) {
            return *(const half8_t *)(a.W + (int64_t)(n0 + cc) * a.K + k);
        } else {
            half8_t h;
#pragma unroll
            for (int j = 0; j < 8; ++j) h[j] = __builtin_bit_cast(_Float16, a.W[(k + j) * a.N + n0 + cc]);
            return h;
        }
    };

    // One ratio leaves nothing to search: its scale stands unless its error is
    // not below infinity, that is unless a value is not finite (of finite fp16
    // values no K can sum up to that).  Zero times each value finds those during
    // the pass for max|v|: with one ratio three of four lanes would repeat the
    // sums of the first (28672 x 8192 at g = 256: 437 us with them, 301 now).
    const bool search = a.n_ratios > 1;
    float zero = 0.0f;  // NaN once a value is not finite
    float amax = 0.0f;  // of this lane's share: the order does not matter
    for (int i = wave * 4 + (lane >> 4); i < chunks * 16; i += waves * 4) {
        const half8_t h = load8(i >> 4, i & 15, c);
#pragma unroll
        for (int j = 0; j < 8; ++j) amax = __builtin_fmaxf(amax, __builtin_fabsf((float)h[j]));
        if (!search) {
#pragma unroll
            for (int j = 0; j < 8; ++j) zero = __builtin_fmaf((float)h[j], 0.0f, zero);
        }
    }
    amax = __builtin_fmaxf(amax, __shfl_xor(amax, 16));
    amax = __builtin_fmaxf(amax, __shfl_xor(amax, 32));
    if (lane < kCols) shared_max[wave][lane] = amax;
    __syncthreads();
    for (int w = 0; w < waves; ++w) amax = __builtin_fmaxf(amax, shared_max[w][c]);

    // The search: this lane's ratio (the last wave's spare lanes repeat the last).
    const int mine = wave * 4 + (lane >> 4);
    const int ratio = mine < a.n_ratios ? mine : a.n_ratios - 1;
    const float sf = (float)scale_of(a.ratios[ratio], amax);
    const float inv = sf == 0.0f ? 0.0f : 1.0f / sf;
    float err = zero;
    auto fill = [&](int ch, int slot) {
        for (int i = threadIdx.x; i < 16 * kCols; i += blockDim.x)
            *(half8_t *)&chunk[slot][(i & 15) * kPitch + (i >> 4) * 8] = load8(ch, i >> 4, i & 15);
    };
    if (search) {
        fill(0, 0);
        __syncthreads();
    } else {  // one wave
        err += __shfl_xor(err, 16);
        err += __shfl_xor(err, 32);
    }
    for (int ch = 0; ch < chunks && search; ++ch) {
        if (ch + 1 < chunks) fill(ch + 1, (ch + 1) & 1);
#pragma unroll 4
        for (int o = 0; o < 16; ++o) {
            const half8_t h = *(const half8_t *)&chunk[ch & 1][c * kPitch + o * 8];
#pragma unroll
            for (int j = 0; j < 8; ++j) err = error_term(err, (float)h[j], inv, sf);
        }
        __syncthreads();
    }
    if (mine < a.n_ratios) errs[mine][c] = err;
    __syncthreads();

    float best_err = __builtin_inff();
    _Float16 best = (_Float16)0.0f;
    for (int i = 0; i < a.n_ratios; ++i) {
        if (errs[i][c] < best_err) {
            best_err = errs[i][c];
            best = scale_of(a.ratios[i], amax);
        }
    }
    const float bs = (float)best;
    const float binv = bs == 0.0f ? 0.0f : 1.0f / bs, on = bs == 0.0f ? 0.0f : 1.0f;
    const int n = n0 + c, lg = lane >> 4;
    for (int ch = wave; ch < chunks; ch += waves) {
        if constexpr (LINEAR) {
            u32x4_t word;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const half8_t h = load8(ch, 4 * t + lg, c);
                word[t] = pack_word([&](int j) { return code_of((float)h[j], binv); }, on);
            }
            uint32_t *w = (uint32_t *)a.q + (((int64_t)(n >> 6) * (a.K / 128) + k0 / 128 + ch) * 4 + ((n >> 4) & 3)) * 256;
            *(u32x4_t *)(w + lane * 4) = word;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const half8_t h = load8(ch, 4 * t + lg, c);
                uint8_t *qc = a.q + (k0 + ch * 128 + 32 * t + 8 * lg) * a.N + n;
#pragma unroll
                for (int j = 0; j < 8; ++j) qc[(int64_t)j * a.N] = (uint8_t)(int)__builtin_fmaf(code_of((float)h[j], binv), on, 8.0f);
            }
        }
    }
    if (wave == 0 && lane < kCols) {
        const int64_t at = LINEAR ? packed_scale_index(gr, n, a.K / a.g) : (int64_t)gr * a.N + n;
        a.s[at] = __builtin_bit_cast(uint16_t, best);
    }
}

}  // namespace

hipError_t launch_quantize(const uint16_t *W, int K, int N, int g, const float *ratios, int n_ratios, bool linear,
                           void *q, uint16_t *s, hipStream_t stream)
{
    QuantArgs a;
    a.W = W;
    a.q = (uint8_t *)q;
    a.s = s;
    a.K = K;
    a.N = N;
    a.g = g;
    a.n_ratios = n_ratios;
    for (int i = 0; i < kMaxQuantRatios; ++i) a.ratios[i] = i < n_ratios ? ratios[i] : 0.0f;
    if (g == 128) {
        const dim3 grid((unsigned)((N + 255) / 256), (unsigned)(K / g));
        if (linear)
            hipLaunchKernelGGL(quantize128_kernel<true>, grid, dim3(256), 0, stream, a);
        else
            hipLaunchKernelGGL(quantize128_kernel<false>, grid, dim3(256), 0, stream, a);
    } else {
        const dim3 grid((unsigned)(N / kCols) * (unsigned)(K / g));
        const dim3 block(64u * (unsigned)((n_ratios + 3) / 4));
        if (linear)
            hipLaunchKernelGGL(quantize_group_kernel<true>, grid, block, 0, stream, a);
        else
            hipLaunchKernelGGL(quantize_group_kernel<false>, grid, block, 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace marlin
