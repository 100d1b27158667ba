// Offline repack of int4 codes and fp16 scales into the order the GEMM
// streams them (Section 3.4: "Maximizing Loading Bandwidth",
// "Dequantization and Tensor Cores", "Groups and Instruction Ordering").
//
// Weight words (uint32), c = 64-column tile, ku = 128-row block, nb = 16-column
// block, l = lane 0..63, t = 0..3:
//   word (((c*KU + ku)*4 + nb)*64 + l)*4 + t holds column n = 64c + 16nb + l%16,
//   rows k = 128ku + 32t + 8(l/16) + j (j = 0..7), code j in nibble
//   (j >> 1) + 4(j & 1).
// The nibble order puts codes j and j+1 sixteen bits apart, so one mask (and
// an or with the magic number) yields two fp16 values at once (dequant_sub in
// gemm.hip, dequant_magic in device.h).
//
// Scales (fp16), r = scale row, lg = n-row group of the MFMA output, i = 0..3:
//   index (((c*G + r)*4 + lg)*4 + nb)*4 + i holds s[r][64c + 16nb + 4lg + i],
// so the 16 scales one output lane needs for a 64-column tile are contiguous.
#include <hip/hip_runtime.h>

#include "internal.h"

namespace marlin {
namespace {

__device__ __forceinline__ int nibble_of(int j) { return (j >> 1) + 4 * (j & 1); }

// A thread takes four adjacent columns over the 32 rows 32t + 8lg + j (t, j) of
// one 128-row block: a row is one dword of four codes, so 16 lanes read 64
// bytes of a row and a wave four octets of rows, and the thread's words are four
// 16-byte vectors (t = 0..3) of adjacent lanes of the packed layout.  Rows j and
// j + 2 share a byte (v_lshl_or), then a 4 x 4 byte transpose gives the columns'
// words.  Bound by memory: 8192 x 28672 in 89 us packing, 90 unpacking (one
// thread per word, eight byte accesses each: 177 and 260).
// (q may have any alignment: callers pass views of larger buffers)
__device__ __forceinline__ uint32_t load_codes(const uint8_t *p)
{
    uint32_t v;
    __builtin_memcpy(&v, p, 4);
    return v;
}

struct PackItem {
    int64_t src;  // byte index of row 8lg of the block, first column
    int64_t dst;  // word index of the first column's t = 0
};

__device__ __forceinline__ PackItem pack_item(int64_t item, int N, int KU)
{
    const int n4 = (int)(item & 15);         // four columns of the 64
    const int lg = (int)((item >> 4) & 3);
    const int64_t unit = item >> 6;          // ku fastest over column tiles: consecutive units read adjacent bytes
    const int tiles = N / 64;
    const int c = (int)(unit % tiles);
    const int ku = (int)(unit / tiles);
    const int n = 4 * n4;
    return {((int64_t)ku * 128 + 8 * lg) * N + 64 * c + n,
            ((((int64_t)c * KU + ku) * 4 + (n >> 4)) * 64 + lg * 16 + (n & 15)) * 4};
}

__global__ void __launch_bounds__(256) pack_weights_kernel(const uint8_t *__restrict__ q, int K, int N,
                                                           uint32_t *__restrict__ w)
{
    const int64_t items = (int64_t)K * N / 128;
    for (int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; item < items;
         item += (int64_t)gridDim.x * blockDim.x) {
        const PackItem it = pack_item(item, N, K / 128);
        uint32_t d[4][8];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j) d[t][j] = load_codes(q + it.src + (int64_t)(32 * t + j) * N);
        uint32_t word[4][4];  // [column][t]
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            constexpr uint32_t m = 0x0F0F0F0Fu;
            // byte c: codes (j, j + 2) of column c in its low and high nibble
            const uint32_t x = (d[t][0] & m) | (d[t][2] & m) << 4, y = (d[t][4] & m) | (d[t][6] & m) << 4;
            const uint32_t u = (d[t][1] & m) | (d[t][3] & m) << 4, v = (d[t][5] & m) | (d[t][7] & m) << 4;
            const uint32_t xy0 = __builtin_amdgcn_perm(y, x, 0x05010400u), xy1 = __builtin_amdgcn_perm(y, x, 0x07030602u);
            const uint32_t uv0 = __builtin_amdgcn_perm(v, u, 0x05010400u), uv1 = __builtin_amdgcn_perm(v, u, 0x07030602u);
            word[0][t] = __builtin_amdgcn_perm(uv0, xy0, 0x05040100u);
            word[1][t] = __builtin_amdgcn_perm(uv0, xy0, 0x07060302u);
            word[2][t] = __builtin_amdgcn_perm(uv1, xy1, 0x05040100u);
            word[3][t] = __builtin_amdgcn_perm(uv1, xy1, 0x07060302u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *(uint4 *)(w + it.dst + 4 * i) = make_uint4(word[i][0], word[i][1], word[i][2], word[i][3]);
    }
}

__global__ void __launch_bounds__(256) unpack_weights_kernel(const uint32_t *__restrict__ w, int K, int N,
                                                             uint8_t *__restrict__ q)
{
    const int64_t items = (int64_t)K * N / 128;
    for (int64_t item = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; item < items;
         item += (int64_t)gridDim.x * blockDim.x) {
        const PackItem it = pack_item(item, N, K / 128);
        uint32_t word[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = *(const uint4 *)(w + it.dst + 4 * i);
            word[i][0] = v.x;
            word[i][1] = v.y;
            word[i][2] = v.z;
            word[i][3] = v.w;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            constexpr uint32_t m = 0x0F0F0F0Fu;
            const uint32_t xy0 = __builtin_amdgcn_perm(word[1][t], word[0][t], 0x05010400u);
            const uint32_t uv0 = __builtin_amdgcn_perm(word[1][t], word[0][t], 0x07030602u);
            const uint32_t xy1 = __builtin_amdgcn_perm(word[3][t], word[2][t], 0x05010400u);
            const uint32_t uv1 = __builtin_amdgcn_perm(word[3][t], word[2][t], 0x07030602u);
            // xy: bytes x0 x1 y0 y1 of two columns; join the pairs
            const uint32_t x = __builtin_amdgcn_perm(xy1, xy0, 0x05040100u), y = __builtin_amdgcn_perm(xy1, xy0, 0x07060302u);
            const uint32_t u = __builtin_amdgcn_perm(uv1, uv0, 0x05040100u), v = __builtin_amdgcn_perm(uv1, uv0, 0x07060302u);
            const uint32_t d[8] = {x & m, u & m, (x >> 4) & m, (u >> 4) & m, y & m, v & m, (y >> 4) & m, (v >> 4) & m};
#pragma unroll
            for (int j = 0; j < 8; ++j) __builtin_memcpy(q + it.src + (int64_t)(32 * t + j) * N, &d[j], 4);
        }
    }
}

// dir = 0: natural [G][N] -> packed; dir = 1: packed -> natural.
__global__ void permute_scales_kernel(const uint16_t *__restrict__ src, int N, int G, int dir,
                                      uint16_t *__restrict__ dst)
{
    const int64_t total = (int64_t)G * N;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(idx & 3);
        const int nb = (int)((idx >> 2) & 3);
        const int lg = (int)((idx >> 4) & 3);
        const int64_t cr = idx >> 6;  // c*G + r
        const int r = (int)(cr % G);
        const int c = (int)(cr / G);
        const int64_t nat = (int64_t)r * N + 64 * c + 16 * nb + 4 * lg + i;
        if (dir == 0)
            dst[idx] = src[nat];
        else
            dst[nat] = src[idx];
    }
}

// ---- 2:4 sparse weights (Section 4) ----
// Unit (c, ku) = 64-column tile c, 128-row block ku, at word (c*KU + ku)*768:
//   codes, 512 words: word ((d >> 2)*64 + l)*4 + (d & 3), d = 2*nb + h, holds
//     the 8 kept codes of column n = 64c + 16nb + l%16 in rows
//     128ku + 64h + 16(l/16) + [0, 16): group g = 0..3 of 4 rows keeps codes
//     j = 2g and 2g + 1 (in increasing row order), code j in nibble
//     (j >> 1) + 4(j & 1);
//   metadata, 256 words: word 512 + l*4 + nb holds, at bits 16h + 4g + 2t,
//     the row (0..3) within group g of kept code 2g + t.
// Kept rows are the first two rows of the group whose code is not 8 (weight
// not zero); a group with fewer is completed with its lowest rows of code 8,
// and the pair is kept in increasing row order.
__global__ void pack_sparse_kernel(const uint8_t *__restrict__ q, int K, int N, uint32_t *__restrict__ w)
{
    const int64_t items = (int64_t)K * N / 32;  // (unit, lane, column block)
    const int KU = K / 128;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < items;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int nb = (int)(idx & 3);
        const int l = (int)((idx >> 2) & 63);
        const int64_t unit = idx >> 8;  // c*KU + ku
        const int ku = (int)(unit % KU);
        const int c = (int)(unit / KU);
        const int n = 64 * c + 16 * nb + (l & 15);
        uint32_t meta = 0;
        uint32_t *uw = w + unit * 768;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t word = 0;
            const int kbase = 128 * ku + 64 * h + 16 * (l >> 4);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint32_t code[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) code[r] = q[(int64_t)(kbase + 4 * g + r) * N + n] & 0xFu;
                int p[2] = {-1, -1}, np = 0;
                for (int r = 0; r < 4 && np < 2; ++r)
                    if (code[r] != 8u) p[np++] = r;
                for (int r = 0; r < 4 && np < 2; ++r)
                    if (r != p[0]) p[np++] = r;
                if (p[0] > p[1]) {
                    const int t = p[0];
                    p[0] = p[1];
                    p[1] = t;
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int j = 2 * g + t;
                    word |= code[p[t]] << (4 * nibble_of(j));
                    meta |= (uint32_t)p[t] << (16 * h + 4 * g + 2 * t);
                }
            }
            const int d = 2 * nb + h;
            uw[((d >> 2) * 64 + l) * 4 + (d & 3)] = word;
        }
        uw[512 + l * 4 + nb] = meta;
    }
}

__global__ void unpack_sparse_kernel(const uint32_t *__restrict__ w, int K, int N, uint8_t *__restrict__ q)
{
    const int64_t items = (int64_t)K * N / 32;
    const int KU = K / 128;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < items;
         idx += (int64_t)gridDim.x * blockDim.x) {
        const int nb = (int)(idx & 3);
        const int l = (int)((idx >> 2) & 63);
        const int64_t unit = idx >> 8;
        const int ku = (int)(unit % KU);
        const int c = (int)(unit / KU);
        const int n = 64 * c + 16 * nb + (l & 15);
        const uint32_t *uw = w + unit * 768;
        const uint32_t meta = uw[512 + l * 4 + nb];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int d = 2 * nb + h;
            const uint32_t word = uw[((d >> 2) * 64 + l) * 4 + (d & 3)];
            const int kbase = 128 * ku + 64 * h + 16 * (l >> 4);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint8_t out[4] = {8, 8, 8, 8};
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int j = 2 * g + t;
                    const int r = (int)((meta >> (16 * h + 4 * g + 2 * t)) & 3u);
                    out[r] = (uint8_t)((word >> (4 * nibble_of(j))) & 0xFu);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) q[(int64_t)(kbase + 4 * g + r) * N + n] = out[r];
            }
        }
    }
}

int blocks_for(int64_t work, int threads)
{
    int64_t b = (work + threads - 1) / threads;
    if (b > 65536) b = 65536;
    return (int)(b < 1 ? 1 : b);
}

}  // namespace

hipError_t launch_pack(const uint8_t *q, const uint16_t *s, int K, int N, int G,
                       uint32_t *w_packed, uint16_t *s_packed, hipStream_t stream)
{
    const int threads = 256;
    const int64_t items = (int64_t)K * N / 128;
    hipLaunchKernelGGL(pack_weights_kernel, dim3(blocks_for(items, threads)), dim3(threads), 0,
                       stream, q, K, N, w_packed);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(permute_scales_kernel, dim3(blocks_for((int64_t)G * N, threads)),
                       dim3(threads), 0, stream, s, N, G, 0, s_packed);
    return hipGetLastError();
}

hipError_t launch_unpack(const uint32_t *w_packed, const uint16_t *s_packed, int K, int N,
                         int G, uint8_t *q, uint16_t *s, hipStream_t stream)
{
    const int threads = 256;
    const int64_t items = (int64_t)K * N / 128;
    hipLaunchKernelGGL(unpack_weights_kernel, dim3(blocks_for(items, threads)), dim3(threads), 0,
                       stream, w_packed, K, N, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(permute_scales_kernel, dim3(blocks_for((int64_t)G * N, threads)),
                       dim3(threads), 0, stream, s_packed, N, G, 1, s);
    return hipGetLastError();
}

hipError_t launch_pack_sparse(const uint8_t *q, const uint16_t *s, int K, int N, int G, uint32_t *w_packed,
                              uint16_t *s_packed, hipStream_t stream)
{
    const int threads = 256;
    const int64_t items = (int64_t)K * N / 32;
    hipLaunchKernelGGL(pack_sparse_kernel, dim3(blocks_for(items, threads)), dim3(threads), 0, stream, q, K, N,
                       w_packed);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(permute_scales_kernel, dim3(blocks_for((int64_t)G * N, threads)), dim3(threads), 0, stream,
                       s, N, G, 0, s_packed);
    return hipGetLastError();
}

hipError_t launch_unpack_sparse(const uint32_t *w_packed, const uint16_t *s_packed, int K, int N, int G,
                                uint8_t *q, uint16_t *s, hipStream_t stream)
{
    const int threads = 256;
    const int64_t items = (int64_t)K * N / 32;
    hipLaunchKernelGGL(unpack_sparse_kernel, dim3(blocks_for(items, threads)), dim3(threads), 0, stream, w_packed,
                       K, N, q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(permute_scales_kernel, dim3(blocks_for((int64_t)G * N, threads)), dim3(threads), 0, stream,
                       s_packed, N, G, 1, s);
    return hipGetLastError();
}

}  // namespace marlin
