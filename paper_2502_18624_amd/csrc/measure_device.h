// Device and host helpers shared by the measurement kernels' translation units.
#pragma once

#include <cstdlib>

#include "common.h"

namespace mcl {

__device__ __forceinline__ uint32_t pick(const uint4& v, int d)
{
    return d == 0 ? v.x : d == 1 ? v.y : d == 2 ? v.z : v.w;
}

// acc + (number of set bits of x) as one v_bcnt_u32_b32.  Written out, sums
// of several bit counts are re-associated into separate counts and
// three-input adds.
__device__ __forceinline__ uint32_t bcnt_acc(uint32_t x, uint32_t acc)
{
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

// a where m is set, else b (one v_bfi_b32 or v_bitop3_b32).
__device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));

// c + a b^T for 16 rows each of a and b, 128 fp4 numbers a row: lane
// (m = lane & 15, h = lane >> 4) holds numbers 32 h .. 32 h + 31 of row m, and
// c[i] of lane (j, h) belongs to row 4 h + i of a and row j of b.
__device__ __forceinline__ v4f mfma_f4(const uint4& a, const uint4& b, v4f c)
{
    const v8i va = {(int)a.x, (int)a.y, (int)a.z, (int)a.w, 0, 0, 0, 0};
    const v8i vb = {(int)b.x, (int)b.y, (int)b.z, (int)b.w, 0, 0, 0, 0};
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(va, vb, c, 4, 4, 0, 0, 0, 0);
}

// 16 columns by 32 rows of staged fp4 cells as an operand, 32 rows from each
// lane group: `cells` is the lane's row (lane & 15 of its group's 16) at the
// columns' 8 bytes, the other 16 rows `half` bytes on.  Lane m of a group gets
// column m.
__device__ __forceinline__ uint4 columns16(char* cells, int half)
{
    typedef __attribute__((address_space(3))) v2i* lp;
    const v2i r0 = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lp)cells);
    const v2i r1 = __builtin_amdgcn_ds_read_tr4_b64_v2i32((lp)(cells + half));
    return make_uint4((uint32_t)r0.x, (uint32_t)r0.y, (uint32_t)r1.x, (uint32_t)r1.y);
}

// 32 one-bit cells as fp4 numbers 0 and 1 (bit 1 of a nibble), each block of
// 16 cells in two words: cells 0, 4, 8, 12, 1, 5, 9, 13 and 2, 6, .., 15.
__device__ __forceinline__ uint4 expand(uint32_t w)
{
    const uint32_t C = 0x22222222u;
    const uint32_t e0 = (w << 1) & C, e1 = w & C, e2 = (w >> 1) & C, e3 = (w >> 2) & C;
    return make_uint4(__builtin_amdgcn_perm(e1, e0, 0x05040100u), __builtin_amdgcn_perm(e3, e2, 0x05040100u),
                      __builtin_amdgcn_perm(e1, e0, 0x07060302u), __builtin_amdgcn_perm(e3, e2, 0x07060302u));
}

// A 4-bit word with only the bits that define a spin: Ising bit 1 (s = +1
// where set), Blume-Capel bit 0 (s = 0 where set), else bit 1.  `bad`
// collects the bits of cells that hold no spin (Blume-Capel: bit 1 of `both`
// too, set where bits 0 and 1 of a cell are).
template <int MODEL>
__device__ __forceinline__ uint32_t clean(uint32_t w, uint32_t& bad, uint32_t& both)
{
    if (MODEL == 0) {
        bad |= w & 0xDDDDDDDDu;
        return w & 0x22222222u;
    }
    const uint32_t up = w << 1;
    bad |= w & 0xCCCCCCCCu;
    both |= w & up;
    return (w & ~up & 0x22222222u) | (w & 0x11111111u);
}

// Optional cap on the workgroups of the measurement kernels that split their
// work freely (B/M/Q pass, measurement pass, sampled x rows): the environment
// variable MCL_MEASURE_GRID, read at every launch.  It changes how the work
// is split over workgroups, never the sums; a test uses it to give each
// workgroup several units, tasks and rows at small L.
inline uint32_t measure_grid_cap(uint32_t want)
{
    if (const char* e = std::getenv("MCL_MEASURE_GRID")) {
        const long long v = std::atoll(e);
        if (v > 0 && (uint64_t)v < want) return (uint32_t)v;
    }
    return want;
}

}  // namespace mcl
