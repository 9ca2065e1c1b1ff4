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
