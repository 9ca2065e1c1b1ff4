// Small lattices, many sweeps, one launch (gfx950): a workgroup holds both
// colour planes of its lattice in LDS and runs every sweep of the call on
// them, reading and writing the lattice in memory once.
//
// A half-sweep of a small lattice as a launch of its own is bound by latency:
// the launch, the loads of a thread's rows and their chain of row steps (L =
// 256: 4.4 us for 2^15 updates, which are 0.012 us of the chip's VALU work).
// Here a half-sweep costs a barrier and its work on one compute unit, bound by
// VALU issue; the draws are keyed by (seed, sweep, site), so the lattice is
// the same.  512 replicas of L = 256, 16 sweeps: 285 us, 78% of the VALU rate
// (the launches per half-sweep took 1190, or 580 with bands short enough to
// fill their tiles).
#include <algorithm>

#include "internal.h"
#include "sweep_device.h"

namespace mcl {
namespace {

// Threads of a workgroup: 1024 while a compute unit gets one workgroup at
// most, else 512, so that two share it and one works while the other waits at
// its barrier (1024 replicas of L = 256, 16 sweeps: 670 us, with 1024 threads
// 750).
constexpr uint32_t kMaxThreads = 1024;

// LDS: the two planes, then the model's table.
template <int MODEL>
__device__ __forceinline__ void run_resident(char* lds, uint32_t* planes, uint32_t L, uint32_t t, uint32_t n,
                                             uint32_t k0, uint32_t k1, uint32_t T4, uint32_t T8, const uint2* tab,
                                             const uint2* B, const uint32_t* lut, uint32_t kmax)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    const uint32_t rowB = (L >> 4) * CB, Q = rowB >> 4, planeB = L * rowB;
    uint4* cells = reinterpret_cast<uint4*>(lds);
    uint4* mem = reinterpret_cast<uint4*>(planes);
    for (uint32_t i = threadIdx.x; i < planeB / 8; i += blockDim.x) cells[i] = mem[i];
    __syncthreads();
    // (both sides' neighbour words and a select per word: one copy of the
    // update's code, and L = 64 has rows of both parities in its one wave)
    const uint32_t vecs = Q * L;
    const uint32_t magic = 0xFFFFFFFFu / Q + 1;             // v / Q = high word of v magic (v Q < 2^32; Q > 1)
    for (uint32_t s = 0; s < n; ++s, ++t)
        for (uint32_t c = 0; c < 2; ++c) {
            char* own = lds + c * planeB;
            const char* oth = lds + (1 - c) * planeB;
            for (uint32_t v = threadIdx.x; v < vecs; v += blockDim.x) {
                const uint32_t y = Q == 1 ? v : __umulhi(v, magic), q = v - y * Q;
                const char* row = oth + y * rowB;
                const char* up = oth + (y == 0 ? L - 1 : y - 1) * rowB;
                const char* dn = oth + (y + 1 == L ? 0 : y + 1) * rowB;
                uint4* at = reinterpret_cast<uint4*>(own + y * rowB) + q;
                const uint4 src = *at, a = dev::load_row(up, 16 * q), b = dev::load_row(dn, 16 * q);
                const uint4 mid = dev::load_row(row, 16 * q);
                const bool odd = ((y + c) & 1u) != 0;
                const uint32_t side = odd ? (q + 1 == Q ? 0u : 16 * q + 16) : (q == 0 ? rowB : 16 * q) - 4;
                const uint32_t halo = *reinterpret_cast<const uint32_t*>(row + side);
                const uint32_t kv = y * (L >> 1) + (128 / CB) * q;              // in-colour index of cell 0
                if (MODEL == 0) {
                    *at = dev::ising_vec<0>(src, a, b, mid, halo, odd, kv >> 2, 0u, t, c, k0, k1, 0u, T4, T8);
                } else if (MODEL == 2) {
                    *at = dev::lut_vec<0>(src, a, b, mid, halo, odd, kv, t, c, k0, k1, 0u, B, lut, T8, kmax);
                } else {
                    const Philox4 p = philox4x32_10(kv >> 7, 0u, t, 2u + c, k0, k1);
                    *at = dev::bc_vec<0>(src, a, b, mid, halo, odd, kv >> 2, 0u, philox_word(p, (int)((kv >> 5) & 3)), t, c,
                                         k0, k1, 0u, tab);
                }
            }
            __syncthreads();
        }
    for (uint32_t i = threadIdx.x; i < planeB / 8; i += blockDim.x) mem[i] = cells[i];
}

// LDS tables of the models of a launch.
struct ResidentLds {
    dev::BCLds bc;
    uint32_t lut[16];
};

template <int MODEL>
__device__ __forceinline__ void resident(ResidentLds& tabs, const GroupDesc& d, uint32_t t, uint32_t n,
                                         const LutTable& lt)
{
    extern __shared__ __align__(16) char lds[];
    const uint32_t L = d.L;
    uint2* B = reinterpret_cast<uint2*>(lds + (size_t)L * L / 8);        // (1-bit: after 2 planes of L^2 / 16 bytes)
    if (MODEL == 2) {
        if (threadIdx.x < 16) tabs.lut[threadIdx.x] = lt.T[threadIdx.x];
        for (uint32_t b = threadIdx.x; b < (uint32_t)dev::kLutBuckets; b += blockDim.x) {
            const uint64_t A = dev::lut_bucket_addend(lt.T, lt.kmax, b);
            B[b] = make_uint2((uint32_t)A, (uint32_t)(A >> 32));
        }
    }
    run_resident<MODEL>(lds, d.plane0, L, t, n, d.k0, d.k1, d.T4, MODEL == 2 ? lt.T[8] : d.T8, tabs.bc.e, B, tabs.lut,
                        lt.kmax);
}

// One lattice, its tables passed by value.
template <int MODEL>
__global__ __launch_bounds__(kMaxThreads) void resident_kernel(GroupDesc d, uint32_t n, BCTable bc, LutTable lt)
{
    __shared__ ResidentLds tabs;
    if (MODEL == 1) dev::load_bc_table(tabs.bc, bc);
    resident<MODEL>(tabs, d, d.t0, n, lt);
}

// Sweeps [s0, min(s1, n)) of one descriptor per workgroup, any mix of models:
// one launch, so that all their workgroups share the chip.
__global__ __launch_bounds__(kMaxThreads) void group_resident_kernel(const GroupDesc* __restrict__ desc, uint32_t s0,
                                                                     uint32_t s1, const uint2* __restrict__ bc_tables,
                                                                     const LutRec* __restrict__ luts)
{
    __shared__ ResidentLds tabs;
    GroupDesc d = desc[blockIdx.x];
    d.T4 = __builtin_amdgcn_readfirstlane(d.T4);
    d.T8 = __builtin_amdgcn_readfirstlane(d.T8);
    const uint32_t end = min(s1, d.n);
    if (s0 >= end) return;
    LutTable lt{};
    if (d.model == 0u) {
        resident<0>(tabs, d, d.t0 + s0, end - s0, lt);
    } else if (d.model == 1u) {
        dev::load_bc_table(tabs.bc, bc_tables + (size_t)d.tab * 96u);
        resident<1>(tabs, d, d.t0 + s0, end - s0, lt);
    } else {
        const LutRec* rec = luts + d.tab;
#pragma unroll
        for (int k = 0; k < 16; ++k) lt.T[k] = __builtin_amdgcn_readfirstlane(rec->T[k]);
        lt.kmax = __builtin_amdgcn_readfirstlane(rec->kmax);
        resident<2>(tabs, d, d.t0 + s0, end - s0, lt);
    }
}

// No more threads than a plane has 16-byte vectors, in whole waves.
uint32_t threads_of(int64_t vectors, int64_t most)
{
    return (uint32_t)std::max<int64_t>(64, std::min<int64_t>(most, (vectors + 63) / 64 * 64));
}

template <class K, class... A>
hipError_t go(K kernel, uint32_t grid, uint32_t threads, size_t lds, hipStream_t s, A... args)
{
    if (lds > 32u * 1024u) {
        const hipError_t e =
            hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, s, args...);
    return hipGetLastError();
}

}  // namespace

size_t resident_lds(int model, int64_t L)
{
    return model == 2 ? (size_t)(L * L / 8) + (size_t)kLutBucketBytes : (size_t)(L * L / 2);
}

hipError_t launch_resident(const GroupDesc& d, uint32_t n, const BCTable& bc, const LutTable& lt, hipStream_t s)
{
    const size_t lds = resident_lds((int)d.model, d.L);
    const uint32_t threads = threads_of((int64_t)d.L * d.L / (d.model == 2 ? 256 : 64), kMaxThreads);
    if (d.model == 0) return go(resident_kernel<0>, 1, threads, lds, s, d, n, bc, lt);
    if (d.model == 1) return go(resident_kernel<1>, 1, threads, lds, s, d, n, bc, lt);
    return go(resident_kernel<2>, 1, threads, lds, s, d, n, bc, lt);
}

hipError_t launch_group_resident(const GroupDesc* desc, int count, size_t lds, int64_t vectors, uint32_t s0, uint32_t s1,
                                 const uint2* bc_tables, const LutRec* luts, hipStream_t s)
{
    const uint32_t threads = threads_of(vectors, count > 256 && lds <= 76u * 1024u ? 512 : kMaxThreads);
    return go(group_resident_kernel, (uint32_t)count, threads, lds, s, desc, s0, s1, bc_tables, luts);
}

}  // namespace mcl
