// Spins to and from the host for gfx950: the kernels address pinned host
// memory themselves, so a lattice crosses the link once, as int8 spins, and no
// device memory beside it is needed.  Bound by the link (56 GB/s) and the
// host's own copy out of the pinned buffer.
#include "internal.h"

namespace mcl {
namespace {

// n - 1 in each byte of v (n = 0 .. 15).
__device__ __forceinline__ uint32_t minus_one(uint32_t v) { return ((v | 0x80808080u) - 0x01010101u) ^ 0x80808080u; }

// Bytes k of a, b, c, d as one word.
template <int K>
__device__ __forceinline__ uint32_t bytes4(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    constexpr uint32_t pair = K | (uint32_t)(K + 4) << 8;               // a's byte, b's byte
    const uint32_t lo = __builtin_amdgcn_perm(b, a, pair), hi = __builtin_amdgcn_perm(d, c, pair);
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// 8 bits at bits 0 and 1 of 4-bit cells' place: bit i to bit 1 of nibble i.
__device__ __forceinline__ uint32_t bits_to_cells(uint32_t x)
{
    x &= 0xFFu;
    x = (x | x << 12) & 0x000F000Fu;
    x = (x | x << 6) & 0x03030303u;
    x = (x | x << 3) & 0x11111111u;
    return x << 1;
}

// Rows y0 .. y0 + rows - 1: thread per 16 sites.  The cells of even x are in
// plane y & 1, those of odd x in the other, at the same place.
template <int CB>
__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ planes, uint32_t L, uint32_t y0,
                                                     uint32_t total, uint4* __restrict__ out)
{
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const uint32_t per = L >> 4, r = g / per, i = g - r * per, y = y0 + r;
    const size_t W = (L >> 6) * (CB == 4 ? 4 : 1), plane = (size_t)L * W;
    const uint32_t* row = planes + (size_t)y * W;
    const size_t pe = (y & 1u) ? plane : 0, po = (y & 1u) ? 0 : plane;
    uint32_t e, o;
    if (CB == 4) {
        e = row[pe + i];
        o = row[po + i];
    } else {
        e = bits_to_cells(row[pe + (i >> 2)] >> (8 * (i & 3u)));
        o = bits_to_cells(row[po + (i >> 2)] >> (8 * (i & 3u)));
    }
    const uint32_t e0 = e & 0x0F0F0F0Fu, e1 = (e >> 4) & 0x0F0F0F0Fu, o0 = o & 0x0F0F0F0Fu, o1 = (o >> 4) & 0x0F0F0F0Fu;
    out[g] = make_uint4(minus_one(bytes4<0>(e0, o0, e1, o1)), minus_one(bytes4<1>(e0, o0, e1, o1)),
                        minus_one(bytes4<2>(e0, o0, e1, o1)), minus_one(bytes4<3>(e0, o0, e1, o1)));
}

// The cells n = s + 1 of the even (odd) sites of 16, as nibbles, spins -1, 0, 1.
__device__ __forceinline__ uint32_t cells_of(const uint4& v, int odd)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t n = (w[k] & 0x03030303u) + 0x01010101u;          // s + 1 in the low two bits of each byte
        const uint32_t a = (n >> (8 * odd)) & 3u, b = (n >> (8 * odd + 16)) & 3u;
        r |= (a | b << 4) << (8 * k);
    }
    return r;
}

// The same the other way: thread per word of each plane (16 or 64 sites).
template <int CB>
__global__ __launch_bounds__(256) void pack_kernel(uint32_t* __restrict__ planes, uint32_t L, uint32_t y0, uint32_t total,
                                                   const uint4* __restrict__ in)
{
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const uint32_t W = (L >> 6) * (CB == 4 ? 4 : 1), r = g / W, i = g - r * W, y = y0 + r;
    const size_t plane = (size_t)L * W;
    uint32_t c[2] = {0, 0};
#pragma unroll
    for (int odd = 0; odd < 2; ++odd) {
        if (CB == 4) {
            c[odd] = cells_of(in[g], odd);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // bit 1 of each nibble (s = +1) to 8 adjacent bits
                uint32_t x = (cells_of(in[4 * (size_t)g + k], odd) >> 1) & 0x11111111u;
                x = (x | x >> 3) & 0x03030303u;
                x = (x | x >> 6) & 0x000F000Fu;
                x = (x | x >> 12) & 0xFFu;
                c[odd] |= x << (8 * k);
            }
        }
    }
    uint32_t* row = planes + (size_t)y * W + i;
    row[(y & 1u) ? plane : 0] = c[0];
    row[(y & 1u) ? 0 : plane] = c[1];
}

// A window, thread per site: rows dy0 .. of the window [x0, x0 + w) x [y0, ..).
__global__ __launch_bounds__(256) void window_kernel(const uint32_t* __restrict__ planes, uint32_t L, int cb, uint32_t x0,
                                                     uint32_t y0, uint32_t w, uint32_t total, int8_t* __restrict__ out)
{
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const uint32_t dy = g / w, dx = g - dy * w;
    uint32_t x = x0 + dx, y = y0 + dy;
    x = x >= L ? x - L : x;
    y = y >= L ? y - L : y;
    const size_t W = cb == 4 ? L >> 4 : L >> 6;
    const uint32_t* row = planes + ((x + y) & 1u) * (size_t)L * W + (size_t)y * W;
    const uint32_t i = x >> 1;
    out[g] = cb == 4 ? (int8_t)((int)((row[i >> 3] >> (4 * (i & 7u))) & 0xFu) - 1)
                     : (int8_t)(((row[i >> 5] >> (i & 31u)) & 1u) ? 1 : -1);
}

uint32_t blocks(uint64_t n) { return (uint32_t)((n + 255) / 256); }

}  // namespace

hipError_t launch_unpack(const Geom& g, int64_t y0, int64_t rows, void* out, hipStream_t s)
{
    const uint32_t total = (uint32_t)(rows * (g.L / 16));
    if (g.cb == 4)
        hipLaunchKernelGGL(unpack_kernel<4>, dim3(blocks(total)), dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)y0,
                           total, reinterpret_cast<uint4*>(out));
    else
        hipLaunchKernelGGL(unpack_kernel<1>, dim3(blocks(total)), dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)y0,
                           total, reinterpret_cast<uint4*>(out));
    return hipGetLastError();
}

hipError_t launch_pack(const Geom& g, int64_t y0, int64_t rows, const void* in, hipStream_t s)
{
    const uint32_t total = (uint32_t)(rows * g.W);
    if (g.cb == 4)
        hipLaunchKernelGGL(pack_kernel<4>, dim3(blocks(total)), dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)y0,
                           total, reinterpret_cast<const uint4*>(in));
    else
        hipLaunchKernelGGL(pack_kernel<1>, dim3(blocks(total)), dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)y0,
                           total, reinterpret_cast<const uint4*>(in));
    return hipGetLastError();
}

hipError_t launch_window(const Geom& g, int64_t x0, int64_t y0, int64_t w, int64_t rows, void* out, hipStream_t s)
{
    const uint32_t total = (uint32_t)(rows * w);
    hipLaunchKernelGGL(window_kernel, dim3(blocks(total)), dim3(256), 0, s, g.plane0, (uint32_t)g.L, g.cb, (uint32_t)x0,
                       (uint32_t)y0, (uint32_t)w, total, reinterpret_cast<int8_t*>(out));
    return hipGetLastError();
}

}  // namespace mcl
