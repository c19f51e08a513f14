// Row-major -> tiled serving layout (see bd_tiled.h).  Offline, like the compressor: run once
// per base matrix and once per (tenant, matrix) delta.
#include "bd_device.h"
#include "bd_tiled.h"

namespace bd {

// One thread per 16-byte unit of the tiled base: unit ((rb KT + kt) 8 + v) 64 + l holds
// W[16 rb + l % 16][256 kt + 32 v + 8 (l / 16) .. + 8].
__global__ __launch_bounds__(256) void tile_base_kernel(const uint16_t* __restrict__ w, u32x4* __restrict__ wt,
                                                         const int64_t out, const int64_t in, const int64_t KT,
                                                         const int64_t n_units) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n_units; u += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(u & 63), v = (int)((u >> 6) & 7);
        const int64_t tile = u >> 9, kt = tile % KT, rb = tile / KT;
        const int64_t row = rb * kTileRows + (l & 15), k = kt * kTileK + 32 * v + 8 * (l >> 4);
        u32x4 val = {0u, 0u, 0u, 0u};
        if (row < out && k < in) val = *(const u32x4*)(w + row * in + k);   // in % 8 == 0: the 8 elements are all inside
        wt[u] = val;
    }
}

// Tiled signs: lane slot l = (r, g) of tile (rb, kt) holds 8 bytes, byte v = bits 8 g .. 8 g + 7 of packed word 8 kt + v of
// row 16 rb + r.  Bound by HBM (1/4 byte per element moved in all).  One thread takes one row of one tile: its 8 words in
// two 128-bit loads, a byte transpose in registers, and the 8 bytes of each of the four lane groups out; a wavefront is 16
// rows x 4 neighbouring tiles, so that it reads whole 128-byte lines and writes 128 contiguous bytes per tile and group.
// (One thread per lane slot, four threads each loading the same 8 words one by one, took 17.2 us for 11008 x 4096 where
// this takes 4.6.)  VEC: rows start at 16-byte boundaries (in % 128 == 0); otherwise word by word.
template <bool VEC>
__global__ __launch_bounds__(256) void tile_signs_kernel(const uint32_t* __restrict__ packed, u32x2* __restrict__ st,
                                                          const int64_t out, const int words_per_row, const uint32_t KT,
                                                          const uint32_t n_rows_of_tiles) {
    const uint32_t t = blockIdx.x * 256u + threadIdx.x;   // tiles * 16 < 2^23 (a tiled base is below 4 GiB)
    if (t >= n_rows_of_tiles) return;
    const uint32_t tile = t >> 4, rb = tile / KT, kt = tile - rb * KT;
    const int r = (int)(t & 15);
    const int64_t row = (int64_t)rb * kTileRows + r;
    const int w0 = (int)kt * 8;                           // first word of the row
    uint32_t w[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    if (row < out) {
        const uint32_t* src = packed + row * words_per_row + w0;
        if constexpr (VEC) {                              // groups of 4 words lie inside the row or beyond it
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (w0 + 4 * h < words_per_row) {
                    const u32x4 q = *(const u32x4*)(src + 4 * h);
#pragma unroll
                    for (int i = 0; i < 4; ++i) w[4 * h + i] = q[i];
                }
        } else {
#pragma unroll
            for (int v = 0; v < 8; ++v)
                if (w0 + v < words_per_row) w[v] = src[v];
        }
    }
    u32x2 val[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const u32x4 t = transpose_bytes(u32x4{w[4 * h], w[4 * h + 1], w[4 * h + 2], w[4 * h + 3]});
#pragma unroll
        for (int g = 0; g < 4; ++g) val[g][h] = t[g];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) st[(int64_t)tile * 64 + g * 16 + r] = val[g];
}

// One 16-byte unit of the 8-bit base layout per thread: unit u = ((tile * 4 + i) * 64 + l), bytes [h][e] =
// 128 + q[16 rb + l % 16][256 kt + 32 (2 i + h) + 8 (l / 16) + e]; 128 (q = 0) outside the matrix.
__global__ __launch_bounds__(256) void tile_base_q8_kernel(const int8_t* __restrict__ q, u32x4* __restrict__ wq,
                                                            const int64_t out, const int64_t in, const int64_t KT,
                                                            const int64_t n_units) {
    for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n_units; u += (int64_t)gridDim.x * blockDim.x) {
        const int l = (int)(u & 63), i = (int)((u >> 6) & 3);
        const int64_t tile = u >> 8, kt = tile % KT, rb = tile / KT;
        const int64_t row = rb * kTileRows + (l & 15);
        u32x4 val = {0x80808080u, 0x80808080u, 0x80808080u, 0x80808080u};
        if (row < out) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t k0 = kt * kTileK + 32 * (2 * i + h) + 8 * (l >> 4);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const uint32_t byte = k0 + e < in ? (uint32_t)(uint8_t)(q[row * in + k0 + e] + 128) : 128u;
                    const int pos = 8 * h + e;
                    val[pos >> 2] = (val[pos >> 2] & ~(0xFFu << (8 * (pos & 3)))) | (byte << (8 * (pos & 3)));
                }
            }
        }
        wq[u] = val;
    }
}

// The same, 128-bit loads (q 16-byte aligned), and the padded scales behind the tiles in the same launch.  Bound by HBM.  A
// thread loads 16 bytes of one row at two places 32 apart (k = 64 i + 16 gp and + 32: both slices of unit i for the lane
// groups 2 gp and 2 gp + 1) and stores the two units they make; a wavefront covers 16 rows x 128 bytes, whole lines.
// (Byte by byte: 90.9 us for 11008 x 4096 and 4.8 us more for the scales; this takes 15.6.)
__global__ __launch_bounds__(256) void tile_base_q8_vec_kernel(const int8_t* __restrict__ q, const float* __restrict__ scale,
                                                                u32x4* __restrict__ wq, float* __restrict__ scale_out,
                                                                const int64_t out, const int64_t in, const uint32_t KT,
                                                                const uint32_t n_threads, const uint32_t n_scales) {
    const uint32_t u = blockIdx.x * 256u + threadIdx.x;   // 128 per tile: < 2^26 (a tiled fp16 base is below 4 GiB)
    if (u < n_scales) scale_out[u] = (int64_t)u < out ? scale[u] : 0.0f;   // 16 per row block, fewer than threads
    if (u >= n_threads) return;
    const int r = (int)(u & 15), gp = (int)(u >> 4) & 1, i = (int)(u >> 5) & 3;
    const uint32_t tile = u >> 7, rb = tile / KT, kt = tile - rb * KT;
    const int64_t row = (int64_t)rb * kTileRows + r;
    u32x4 half[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        half[h] = u32x4{0u, 0u, 0u, 0u};
        const int64_t k0 = (int64_t)kt * kTileK + 64 * i + 32 * h;   // in % 32 == 0: a slice is inside the row or beyond it
        if (row < out && k0 < in) half[h] = *(const u32x4*)(q + row * in + k0 + 16 * gp);
#pragma unroll
        for (int d = 0; d < 4; ++d) half[h][d] ^= 0x80808080u;       // q -> q + 128
    }
    u32x4* dst = wq + ((int64_t)tile * 4 + i) * 64 + r;
    dst[(2 * gp) * 16] = u32x4{half[0][0], half[0][1], half[1][0], half[1][1]};
    dst[(2 * gp + 1) * 16] = u32x4{half[0][2], half[0][3], half[1][2], half[1][3]};
}

// scales of the rows of every row block, zero beyond `out`
__global__ __launch_bounds__(256) void tile_scales_kernel(const float* __restrict__ scale, float* __restrict__ dst,
                                                           const int64_t out, const int64_t n_padded) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_padded; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = i < out ? scale[i] : 0.0f;
}

__global__ __launch_bounds__(256) void fill_zero_u16_kernel(uint16_t* __restrict__ p, const int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = 0;
}

static unsigned grid_for(int64_t n, int block) {
    int64_t g = (n + block - 1) / block;
    return (unsigned)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

hipError_t launch_tile_base(const uint16_t* w, int64_t out, int64_t in, uint16_t* wt, hipStream_t st) {
    const int64_t KT = tiled_k_tiles(in), n_units = tiled_row_blocks(out) * KT * (kTileBaseBytes / 16);
    hipLaunchKernelGGL(tile_base_kernel, dim3(grid_for(n_units, 256)), dim3(256), 0, st, w, (u32x4*)wt, out, in, KT, n_units);
    return hipGetLastError();
}

hipError_t launch_tile_signs(const uint32_t* packed, int64_t out, int64_t in, uint32_t* st_out, hipStream_t st) {
    const int64_t KT = tiled_k_tiles(in), n = tiled_row_blocks(out) * KT * kTileRows;
    if (n > (int64_t)1 << 30) return hipErrorInvalidValue;
    if (n == 0) return hipSuccess;
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    const int wpr = (int)(in >> 5);
    if (wpr % 4 == 0)
        hipLaunchKernelGGL(tile_signs_kernel<true>, grid, block, 0, st, packed, (u32x2*)st_out, out, wpr, (uint32_t)KT, (uint32_t)n);
    else
        hipLaunchKernelGGL(tile_signs_kernel<false>, grid, block, 0, st, packed, (u32x2*)st_out, out, wpr, (uint32_t)KT, (uint32_t)n);
    return hipGetLastError();
}

// p[0 .. n) = 0 (a kernel rather than a memset node: safe to capture into a HIP graph)
hipError_t launch_fill_zero_u16(uint16_t* p, int64_t n, hipStream_t st) {
    if (n > 0) hipLaunchKernelGGL(fill_zero_u16_kernel, dim3(grid_for(n, 256)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_tile_base_q8(const int8_t* q, const float* scale, int64_t out, int64_t in, unsigned char* wq, hipStream_t st) {
    const int64_t KT = tiled_k_tiles(in), RB = tiled_row_blocks(out), n_units = RB * KT * (kTileBaseQ8Bytes / 16);
    if (n_units > 0 && ((uintptr_t)q & 15) == 0 && n_units < (int64_t)1 << 30) {   // rows are multiples of 32 bytes
        const int64_t n = RB * KT * 128;
        hipLaunchKernelGGL(tile_base_q8_vec_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, q, scale, (u32x4*)wq,
                           (float*)(wq + RB * KT * kTileBaseQ8Bytes), out, in, (uint32_t)KT, (uint32_t)n, (uint32_t)(RB * kTileRows));
        return hipGetLastError();
    }
    if (n_units > 0)
        hipLaunchKernelGGL(tile_base_q8_kernel, dim3(grid_for(n_units, 256)), dim3(256), 0, st, q, (u32x4*)wq, out, in, KT, n_units);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tile_scales_kernel, dim3(grid_for(RB * kTileRows, 256)), dim3(256), 0, st, scale,
                       (float*)(wq + RB * KT * kTileBaseQ8Bytes), out, RB * kTileRows);
    return hipGetLastError();
}

}  // namespace bd
