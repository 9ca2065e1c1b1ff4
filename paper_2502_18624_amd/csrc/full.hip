// Correlations from every source at every distance r = 33 .. L / 2 (the FULL
// mode beyond the measurement pass), on the matrix cores, for gfx950.
//
// As in the measurement pass (pass.hip) a cell is the fp4 number n / 2 and
// C(r) = 4 P(r) - 2 sum n + L^2; the kernel adds 4 P(r) to Cx and Cy and sum n
// to acc[15], and the host the rest.  A block product of 16 rows (or columns)
// by 16 is useful in all its 256 entries here: entry (i, j) of blocks a and
// a + d has the distance 16 d + j - i.
//
// Along y a wave takes 8 block distances and, at a time, 8 source blocks and
// 128 cells of their rows: 8 + 15 fragments, loaded together straight from
// memory (the lattice is in cache), and 64 products.  Along x a workgroup
// stages 32 rows in LDS, and a wave walks their columns, 4 block distances
// at a time, with the target blocks in a sliding window; an operand holds 32
// rows of one block in each lane group, the groups a quarter of the row apart.
// The two axes are different workgroups of one launch.
//
// 4-bit Ising L = 2112, 1024 distances: 22 us, of which the products alone
// would take 5 (the rest is latency: loads, staging, sums); reading the
// partners of every word from memory for each distance, as lattices that do
// not fit LDS still do (L > 8960), took 1092 us.
#include <algorithm>

#include "internal.h"
#include "measure_device.h"

namespace mcl {
namespace {

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kDistY = 8;           // block distances of a y wave, and its source blocks at a time
constexpr int kDistX = 4;           // block distances of an x wave

// A 32-cell vector as fp4 numbers: 4-bit cells with bit 0 set are 0, the
// others -1 or +1 by bit 1.
template <int CB>
__device__ __forceinline__ uint4 cells32(const char* row, uint32_t v)
{
    if (CB == 1) return expand(reinterpret_cast<const uint32_t*>(row)[v]);
    uint4 w = reinterpret_cast<const uint4*>(row)[v];
    uint32_t unused = 0;
    w.x = clean<1>(w.x, unused, unused);
    w.y = clean<1>(w.y, unused, unused);
    w.z = clean<1>(w.z, unused, unused);
    w.w = clean<1>(w.w, unused, unused);
    return w;
}

// LDS bytes of a staged row: an odd number of 16-byte units, so that 16 rows
// start in different banks.
__host__ __device__ inline uint32_t staged_row(uint32_t L) { return ((L >> 6) | 1u) * 16 + ((L >> 6) & 1u ? 32 : 0); }

template <int CB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void corr_full_kernel(
    const uint32_t* __restrict__ planes, uint32_t L, uint32_t nx, uint32_t per_y, int64_t* __restrict__ Cx,
    int64_t* __restrict__ Cy, int64_t* __restrict__ acc)
{
    extern __shared__ __align__(16) char lds[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 15, h = lane >> 4;
    const uint32_t half = L >> 1, vecs = L >> 6;             // 32-cell vectors of a plane row
    const uint32_t rowB = (L >> 4) * CB;
    const size_t planeB = (size_t)L * rowB;
    const char* base = reinterpret_cast<const char*>(planes);

    if (blockIdx.x >= nx) {
        // along y: workgroup w of the per_y that share block distances d0 .. d0 + 7
        int* sum = reinterpret_cast<int*>(lds);              // distances 16 d0 - 15 .. 16 (d0 + 7) + 15
        constexpr int kSpan = 16 * kDistY + 15;
        for (int i = threadIdx.x; i < kSpan; i += kThreads) sum[i] = 0;
        __syncthreads();
        const uint32_t group = (blockIdx.x - nx) / per_y, part = (blockIdx.x - nx) % per_y;
        const uint32_t d0 = 2 + kDistY * group, blocks = L >> 4;
        const uint32_t chunks = 2 * ((vecs + 3) >> 2), ranges = (blocks + kDistY - 1) / kDistY;
        v4f c[kDistY];
#pragma unroll
        for (int j = 0; j < kDistY; ++j) c[j] = v4f{0.f, 0.f, 0.f, 0.f};
        for (uint32_t task = part * kWaves + wave; task < chunks * ranges; task += per_y * kWaves) {
            const uint32_t chunk = task % chunks, a0 = task / chunks * kDistY;
            const uint32_t p = chunk & 1u, v = 4 * (chunk >> 1) + (uint32_t)h;
            const char* u = base + ((p + (uint32_t)m) & 1u) * planeB + (size_t)m * rowB;       // row m of U_p
            const bool in = v < vecs;
            const auto block = [&](uint32_t b) {
                b = b >= blocks ? b - blocks : b;
                b = b >= blocks ? b - blocks : b;
                return cells32<CB>(u + (size_t)b * 16 * rowB, in ? v : 0u);
            };
            uint4 s[kDistY], t[2 * kDistY - 1];
#pragma unroll
            for (int i = 0; i < kDistY; ++i) s[i] = block(a0 + i);
#pragma unroll
            for (int i = 0; i < 2 * kDistY - 1; ++i) t[i] = block(a0 + d0 + i);
#pragma unroll
            for (int i = 0; i < kDistY; ++i) {
                // (zero past the row's last vector and past the last block)
                if (!in || a0 + i >= blocks) s[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < kDistY; ++j) c[j] = mfma_f4(s[i], t[i + j], c[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < kDistY; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = 16 * j + 15 + m - (4 * h + i);
                if (c[j][i] != 0.f) atomicAdd(&sum[at], (int)(4.f * c[j][i]));
            }
        __syncthreads();
        for (int i = threadIdx.x; i < kSpan; i += kThreads) {
            const uint32_t r = 16 * d0 - 15 + i;
            if (r > 32 && r <= half && sum[i] != 0)
                atomicAdd((unsigned long long*)&Cy[r], (unsigned long long)(long long)sum[i]);
        }
        return;
    }

    // along x: rows 32 blockIdx.x .. + 31, U_p row r at slot 32 p + r
    const uint32_t stride = staged_row(L);
    int* sum = reinterpret_cast<int*>(lds + 64 * stride);    // distances 0 .. half
    for (uint32_t i = threadIdx.x; i <= half; i += kThreads) sum[i] = 0;
    uint32_t total = 0;
    for (uint32_t i = threadIdx.x; i < 64 * vecs; i += kThreads) {
        const uint32_t slot = i / vecs, v = i - slot * vecs, p = slot >> 5, r = slot & 31u;
        const uint4 w = cells32<CB>(base + ((p + r) & 1u) * planeB + (size_t)(32 * blockIdx.x + r) * rowB, v);
        *reinterpret_cast<uint4*>(lds + slot * stride + 16 * v) = w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            total = bcnt_acc(pick(w, d), total);             // n = 2 counts once, n = 1 once
            total = bcnt_acc(pick(w, d) & 0x22222222u, total);
        }
    }
    __syncthreads();
    const uint32_t blocks = L >> 5, last = L >> 6;           // column blocks of a U_p row; largest block distance
    const uint32_t steps = (blocks + 3) >> 2;
    for (uint32_t d0 = 1 + kDistX * (uint32_t)wave; d0 <= last; d0 += kDistX * kWaves) {
        const auto column = [&](int p, uint32_t b) {
            b = b >= blocks ? b - blocks : b;
            return columns16(lds + (32 * p + m) * stride + 8 * b, 16 * stride);
        };
        v4f E[kDistX], A[kDistX], B[kDistX];                 // U_p U_p, U_0 U_1, U_1 U_0
        uint4 T0[kDistX], T1[kDistX];
        const uint32_t b0 = (uint32_t)h * steps;
#pragma unroll
        for (int j = 0; j < kDistX; ++j) {
            E[j] = A[j] = B[j] = v4f{0.f, 0.f, 0.f, 0.f};
            T0[j] = column(0, b0 + d0 + j);
            T1[j] = column(1, b0 + d0 + j);
        }
        for (uint32_t k = 0; k < steps; ++k) {
            uint4 F0 = column(0, b0 + k), F1 = column(1, b0 + k);
            const uint4 N0 = column(0, b0 + k + d0 + kDistX), N1 = column(1, b0 + k + d0 + kDistX);
            if (b0 + k >= blocks) F0 = F1 = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < kDistX; ++j) {
                E[j] = mfma_f4(F0, T0[j], E[j]);
                A[j] = mfma_f4(F0, T1[j], A[j]);
                B[j] = mfma_f4(F1, T0[j], B[j]);
                E[j] = mfma_f4(F1, T1[j], E[j]);
            }
#pragma unroll
            for (int j = 0; j + 1 < kDistX; ++j) {
                T0[j] = T0[j + 1];
                T1[j] = T1[j + 1];
            }
            T0[kDistX - 1] = N0;
            T1[kDistX - 1] = N1;
        }
        const auto cell = [](int j) { return CB == 1 ? 4 * (j & 3) + (j >> 2) : j; };
        const auto add = [&](int r, float v) {
            if (r > 32 && r <= (int)half && v != 0.f) atomicAdd(&sum[r], (int)(4.f * v));
        };
#pragma unroll
        for (int j = 0; j < kDistX; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (d0 + j > last) break;
                const int o = 16 * (int)(d0 + j) + cell(m) - cell(4 * h + i);
                add(2 * o, E[j][i]);
                add(2 * o + 1, A[j][i]);
                add(2 * o - 1, B[j][i]);
            }
    }
    __syncthreads();
    for (uint32_t r = 33 + threadIdx.x; r <= half; r += kThreads)
        if (sum[r] != 0) atomicAdd((unsigned long long*)&Cx[r], (unsigned long long)(long long)sum[r]);
    const int n = wave_sum_i32((int)total);
    if (lane == 0) atomicAdd((unsigned long long*)&acc[15], (unsigned long long)n);
}

size_t full_lds(int64_t L)
{
    return std::max<size_t>((size_t)64 * staged_row((uint32_t)L) + ((size_t)L / 2 + 1) * 4, (16 * kDistY + 15) * 4);
}

}  // namespace

bool full_fits(int64_t L) { return full_lds(L) <= kLdsBytes; }

hipError_t launch_corr_full(const Geom& g, int64_t* Cx, int64_t* Cy, int64_t* acc, hipStream_t s)
{
    const uint32_t L = (uint32_t)g.L;
    if (L < 128 || !full_fits(g.L)) return hipErrorInvalidValue;
    const uint32_t nx = L / 32;
    const uint32_t groups = (L / 32 - 1 + kDistY - 1) / kDistY;     // block distances 2 .. L / 32
    const uint32_t tasks = 2 * ((L / 64 + 3) / 4) * ((L / 16 + kDistY - 1) / kDistY);
    // about two workgroups per CU along y; a wave's products stay far below
    // the 2^22 / 128 that its sums can take
    const uint32_t per_y = std::max<uint32_t>(1, std::min<uint32_t>(512 / groups, (tasks + kWaves - 1) / kWaves));
    const size_t lds = full_lds(g.L);
    const auto go = [&](auto kernel) {
        const hipError_t e = allow_lds(kernel, lds, kLdsBytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(nx + groups * per_y), dim3(kThreads), lds, s, g.plane0, L, nx, per_y, Cx, Cy, acc);
        return hipGetLastError();
    };
    return g.cb == 1 ? go(corr_full_kernel<1>) : go(corr_full_kernel<4>);
}

}  // namespace mcl
