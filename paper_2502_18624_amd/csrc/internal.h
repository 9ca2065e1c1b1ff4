// Host-side declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace mcl {

// Geometry of one lattice in device memory (layout described in common.h).
struct Geom {
    int64_t L;          // linear size, multiple of 64 (256 for 1-bit cells)
    int64_t W;          // 32-bit words per plane row: L / 16 (4-bit cells), L / 64 (1-bit)
    int64_t Q;          // 16-byte vectors per plane row: L / 64 (4-bit cells), L / 256 (1-bit)
    int cb;             // bits per cell: 4 or 1
    uint32_t* plane0;   // colour 0 cells; colour 1 follows at plane0 + L * W
    uint32_t* plane(int c) const { return plane0 + (c ? L * W : 0); }
    int64_t plane_words() const { return L * W; }
};

// Lets launches of a kernel on the current device take `lds` bytes of dynamic
// LDS where that is more than any launch may.  The limit belongs to the kernel,
// so what is set is the most that any of its launches takes: threads that launch
// it for lattices of different sizes at the same time set the same value.
template <class K>
hipError_t allow_lds(K kernel, size_t lds, size_t most)
{
    if (lds <= 32u * 1024u) return hipSuccess;
    if (lds > most) return hipErrorInvalidValue;
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
}
constexpr size_t kLdsBytes = 160 * 1024;    // of a workgroup

// Write the initial state into both planes.
hipError_t launch_init(const Geom& g, int model, int init_state, uint64_t seed, hipStream_t s);

// One colour of one sweep.
struct HalfSweepArgs {
    int color;
    uint32_t t;             // sweep index, or its offset from *tbase when tbase is set
    const uint32_t* tbase;  // device word added to t by the kernel (nullptr: t is absolute)
    uint64_t seed;
    uint32_t T4, T8;        // Ising thresholds (e^{-4 beta}, e^{-8 beta})
    const BCTable* bc;      // Blume-Capel table (host copy, passed by value)
};
hipError_t launch_ising_half(const Geom& g, const HalfSweepArgs& a, hipStream_t s);
// 1-bit Ising with table-driven random bits (W = L/64, Q = L/256 in Geom).
// Bucket table of the 1-bit mode: kLutBucketBytes of device memory, built
// once per beta, read by every half-sweep at that beta.
constexpr int64_t kLutBucketBytes = 4096 * 8;
hipError_t launch_lut_buckets(const LutTable& tab, void* buckets, hipStream_t s);
hipError_t launch_lut_half(const Geom& g, int color, uint32_t t, const uint32_t* tbase, uint64_t seed,
                           const LutTable& tab, const void* buckets, hipStream_t s);
hipError_t launch_bc_half(const Geom& g, const HalfSweepArgs& a, hipStream_t s);
// One device word: *p = v, or *p += v with add (a one-lane kernel, so that
// it can sit in a captured graph).
hipError_t launch_set_word(uint32_t* p, uint32_t v, bool add, hipStream_t s);

// Rows [y0, y0 + rows) to int8 spins in pinned host memory and back, and rows
// y0 .. (periodic, y0 < 2 L) of the window of columns [x0, x0 + w); at most
// 2^31 spins.
hipError_t launch_unpack(const Geom& g, int64_t y0, int64_t rows, void* out, hipStream_t s);
hipError_t launch_pack(const Geom& g, int64_t y0, int64_t rows, const void* in, hipStream_t s);
hipError_t launch_window(const Geom& g, int64_t x0, int64_t y0, int64_t w, int64_t rows, void* out, hipStream_t s);

// Measurement kernels accumulating into int64 device scratch.
// acc layout: [0] B, [1] M (from +1 count minus -1 count), [2] #(+1),
// [3] #(-1), [4] #(0), [5..13] the sigma-h histogram, [14], [15] below; cells
// that are none of the three (corrupted) are L^2 minus the three counts.
constexpr int kAccSlots = 16;
// Before the kernels of a measurement: acc and the nr sums of Cx and Cy to
// zero, and (host_r set) the nr distances from pinned host memory to rdev.
hipError_t launch_begin(int64_t* acc, int64_t* Cx, int64_t* Cy, int nr, int32_t* rdev, const int32_t* host_r,
                        hipStream_t s);
// After them: acc, Cx and Cy, one after the other, to pinned host memory.
hipError_t launch_finish(const int64_t* acc, const int64_t* Cx, const int64_t* Cy, int nr, int64_t* host, hipStream_t s);
// T bits of the sampled columns x = 0 mod 16: for every row y, bit j of its
// word k is [s(16 (32 k + j), y) = +1] (and, Blume-Capel only, a second
// plane of [s != 0] after the first); tbits_words(L) words per row, the L / 16
// bits of a row repeated to fill one word below L = 512 (L is a power of
// two wherever they are used; other L get room for ceil(L / 512) words).
// Word k of row y = 16 b + rho is at k L + rho (L / 16) + b: the rows of one
// residue class follow each other, as the sampled y pass reads them.
// 4-bit Ising lattices from L = 512 on have room after that plane for the
// residue rows of the sampled rows y = 16 b: bit j of word (b tbits_words(L)
// + k) 16 + rho is [s(16 (32 k + j) + rho, y) = +1], read by the sampled x pass.
inline int64_t tbits_words(int64_t L) { return L >= 512 ? (L + 511) / 512 : 1; }
inline int64_t tbits_bytes(int model, int64_t L) { return (model == 2 ? 1 : 2) * L * tbits_words(L) * 4; }
// B, M, Q, counts and the sigma-h histogram into acc, from the cells alone.
hipError_t launch_bmq(const Geom& g, int model, int64_t* acc, hipStream_t s);
// The measurement pass: correlations from every source at r = 0 .. 32 into
// Cx and Cy (33 sums each); with acc set the counts #(+1) [2] and #(0) [4],
// the sigma-h histogram [5 .. 13], and in [14] the number of waves that met a
// cell holding no spin, for which the caller must run launch_bmq instead (acc
// zeroed); with tbits set (L >= 512, a power of two) the T bits and with
// rbits set (4-bit Ising) the residue rows.
hipError_t launch_pass(const Geom& g, int model, int64_t* Cx, int64_t* Cy, int64_t* acc, uint32_t* tbits,
                       uint32_t* rbits, hipStream_t s);
// The T bits of a lattice below L = 512.
hipError_t launch_tbits(const Geom& g, int model, uint32_t* tbits, hipStream_t s);
// Whether measure() takes B/M/Q from the measurement pass when it runs it:
// yes, unless the environment variable MCL_MEASURE_FUSED is 0 (read at every
// call; a test compares the two).
bool bmq_fused();
// Correlations from every source at r = 33 .. L / 2 (Cx, Cy indexed by r):
// adds 4 P(r), P the sum of (n / 2)(n' / 2) over the sources (cells with bit 0
// set counted as n = 1), and sum n to acc[15], so that
// C(r) = what was added - 2 acc[15] + L^2.  Lattices that full_fits() takes.
bool full_fits(int64_t L);
hipError_t launch_corr_full(const Geom& g, int64_t* Cx, int64_t* Cy, int64_t* acc, hipStream_t s);
// Correlations from every source at distances r[0..nr) (any r <= L/2).
hipError_t launch_corr_all(const Geom& g, const int32_t* r_dev, int nr, int64_t* Cx, int64_t* Cy,
                           hipStream_t s);
// Correlations from the sampled sources x = y = 0 (mod 16) at r[0..nr).
struct SampledArgs {
    const int32_t* r;
    int nr;
    int64_t* Cx;
    int64_t* Cy;
    const uint32_t* tbits;
    const uint32_t* rbits = nullptr;    // residue rows (4-bit Ising from L = 512 on), or null
};
// The sampled sources' two passes: x (the lattice's sampled rows, or the
// residue rows when rbits is set) and y (the T bits only).
hipError_t launch_corr_sampled_x(const Geom& g, int model, const SampledArgs& a, hipStream_t s);
hipError_t launch_corr_sampled_y(const Geom& g, int model, const SampledArgs& a, hipStream_t s);

// Batched half-sweep.  One descriptor per replica (64 bytes).  The work of
// a launch is a list of tiles of 256 threads; replica i owns the tiles
// [tile_begin, next replica's tile_begin).  A thread of a tile is one
// 16-byte column vector (32 four-bit or 128 one-bit cells) of one band of
// `rows` rows, as in the one-lattice kernels.
struct GroupDesc {
    uint32_t* plane0;      // the replica's planes (P_1 follows P_0)
    uint32_t L;
    uint32_t rows;         // band rows: even, divides L
    uint32_t t0;           // sweep counter at the start of the call
    uint32_t n;            // sweeps for this replica in this call
    uint32_t k0, k1;       // Philox key (seed)
    uint32_t T4, T8;       // Ising thresholds (4-bit Ising)
    uint32_t tile_begin;   // first tile of this replica in its launch
    uint32_t model;        // 0: Ising 4-bit, 1: Blume-Capel, 2: Ising 1-bit
    uint32_t tab;          // Blume-Capel: index of its 96-entry table; 1-bit: index of its LutRec
    uint32_t pad[3];
};
static_assert(sizeof(GroupDesc) == 64, "descriptor size");

// Table of a 1-bit replica in the batched path: its bucket table (in the
// replica's own device buffer, rebuilt per call) and the 16 clamped
// thresholds with the last index below 2^32.
struct LutRec {
    uint2* buckets;
    uint32_t T[16];
    uint32_t kmax;
    uint32_t pad;
};
static_assert(sizeof(LutRec) == 80, "1-bit record size");

// Models a batched launch may hold (bit m for model m).  A launch whose mask
// has one bit runs that model's path only (and its register budget).
constexpr int kMaskIsing = 1, kMaskBC = 2, kMaskLut = 4;

// One colour of sweep s (+ *sbase when sbase is set) for every replica of
// the list with s < n; grid workgroups (a multiple of 8) walk the `total`
// tiles, those of XCD x the tiles share[x] .. share[x + 1] - 1.  With fewer
// workgroups than tiles they claim tiles from the 16 counter words at ctr,
// which must be zero before the first such launch and are zero again after
// each (nullptr: a fixed walk).
hipError_t launch_group_half(int mask, int color, const GroupDesc* desc, int count, uint32_t total,
                             uint32_t grid, const uint32_t* share, const uint2* bc_tables, const LutRec* luts,
                             uint32_t s, const uint32_t* sbase, uint32_t* ctr, hipStream_t st);
// Lattices that a workgroup holds in LDS (resident_lds bytes of it: both
// planes, and the bucket table of 1-bit cells), in one launch: n sweeps of a
// single lattice with its tables by value, or sweeps [s0, min(s1, n)) of
// `count` descriptors of any models, at most `lds` bytes and `vectors` 16-byte
// vectors of a plane each.
inline size_t resident_lds(int model, int64_t L)
{
    return model == 2 ? (size_t)(L * L / 8) + (size_t)kLutBucketBytes : (size_t)(L * L / 2);
}
hipError_t launch_resident(const GroupDesc& d, uint32_t n, const BCTable& bc, const LutTable& lt, hipStream_t s);
hipError_t launch_group_resident(const GroupDesc* desc, int count, size_t lds, int64_t vectors, uint32_t s0, uint32_t s1,
                                 const uint2* bc_tables, const LutRec* luts, hipStream_t s);
// Up to trapezoid_sweeps() sweeps (0: none) of one lattice in two launches, in
// place, from sweep index t on; at least two.  Worth it for calls of
// trapezoid_least() sweeps or more.
int64_t trapezoid_sweeps(const Geom& g);
int64_t trapezoid_least(const Geom& g);
hipError_t launch_trapezoids(const Geom& g, int model, int64_t sweeps, uint32_t t, uint64_t seed,
                             uint32_t T4, uint32_t T8, const BCTable& bc, const LutTable& lt, const void* buckets,
                             hipStream_t s);
// One half-sweep of a lattice for which half_by_words(), a word per thread
// (1-bit cells without the bucket table).
bool half_by_words(const Geom& g);
hipError_t launch_half_words(const Geom& g, int model, int color, uint32_t t, uint64_t seed, uint32_t T4, uint32_t T8,
                             const BCTable& bc, const LutTable& lt, hipStream_t s);
// Bucket tables of the 1-bit replicas of a batched call.
hipError_t launch_group_lut_buckets(const LutRec* luts, int n, hipStream_t st);

}  // namespace mcl
