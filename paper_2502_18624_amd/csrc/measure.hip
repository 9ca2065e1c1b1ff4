// Measurement kernels for gfx950 beside the measurement pass (pass.hip): B,
// M, Q, counts and the Schwinger-Dyson histogram alone; the correlation sums
// of section 3.3 from every source beyond r = 32 and from the sampled ones.
//
// Energy-like sums.  Every bond of the periodic lattice joins a colour-0 and
// a colour-1 site (L even), so the bond sum B is the sum over colour-0 cells
// of s times the sum of its four neighbours; products of two cells are
// counted eight at a time with popcounts (cell n = s + 1: a product is
// nonzero iff neither cell is 1, and +1 iff bit 1 agrees; Ising cells are
// never 1, so there a word pair needs one xor-and and one popcount).
//
// Correlations (section 3.3).  For a source at (x, y) in plane c:
//   along y the partner (x, y + r) is in plane c ^ (r & 1), row y + r, same
//   in-plane index, so whole words pair up;
//   along x the partner (x + r, y) is in plane c ^ (r & 1) at in-plane index
//   i + m with m = r / 2 (r even) or (r - 1) / 2 + ((y + c) & 1) (r odd), a
//   funnel shift of two neighbouring words.
// The sampled sources (x = y = 0 mod 16) are taken as bits: residue rows
// along x, the T bits along y.
#include <algorithm>
#include <cstdlib>

#include "internal.h"
#include "measure_device.h"

namespace mcl {
namespace {

__global__ __launch_bounds__(256) void begin_kernel(int64_t* __restrict__ acc, int64_t* __restrict__ Cx,
                                                    int64_t* __restrict__ Cy, int nr, int32_t* __restrict__ rdev,
                                                    const int32_t* __restrict__ host_r)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kAccSlots) acc[i] = 0;
    if (i < nr) {
        Cx[i] = Cy[i] = 0;
        if (host_r) rdev[i] = host_r[i];
    }
}

__global__ __launch_bounds__(256) void finish_kernel(const int64_t* __restrict__ acc, const int64_t* __restrict__ Cx,
                                                     const int64_t* __restrict__ Cy, int nr,
                                                     int64_t* __restrict__ host)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kAccSlots) host[i] = acc[i];
    if (i < nr) {
        host[kAccSlots + i] = Cx[i];
        host[kAccSlots + nr + i] = Cy[i];
    }
}

__device__ __forceinline__ uint32_t wrap(uint32_t v, uint32_t n) { return v >= n ? v - n : v; }

// Per-word cell counts: +1 (n = 2), -1 (n = 0), 0 (n = 1); anything else is
// what they leave.  Bit 0 of each nibble carries the test; the mask of the
// other bits is folded into `high`, so each count is one three-input
// logic operation and one bit count.
__device__ __forceinline__ void cell_counts(uint32_t w, uint32_t& np1, uint32_t& nm1, uint32_t& n0)
{
    const uint32_t b1 = w >> 1, high = (w >> 2) | (w >> 3) | 0xEEEEEEEEu;
    np1 = bcnt_acc(b1 & ~w & ~high, np1);
    nm1 = bcnt_acc(~(w | b1 | high), nm1);
    n0 = bcnt_acc(w & ~(b1 | high), n0);
}

// Sum of s * s' over the 8 cell pairs of two words, as (nonzero pairs,
// pairs of opposite sign): the sum is nz - 2 * diff.
__device__ __forceinline__ void pair_counts(uint32_t a, uint32_t b, uint32_t& nz, uint32_t& diff)
{
    const uint32_t z = ~(a | b) & 0x11111111u;
    nz = bcnt_acc(z, nz);
    diff = bcnt_acc(((a ^ b) >> 1) & z, diff);
}

// Cell width traits: 4-bit cells (n = s + 1, 8 per word) and 1-bit cells
// (bit = [s > 0], Ising only, 32 per word).
template <int CB>
struct Cell;

template <>
struct Cell<4> {
    static constexpr int kPerWord = 8;
    static constexpr int kVecShift = 6;     // 16-byte vectors per row = L >> 6
    static constexpr int kWordShift = 4;    // words per row = L >> 4
    static __device__ __forceinline__ void pair(uint32_t a, uint32_t b, uint32_t& nz, uint32_t& diff)
    {
        pair_counts(a, b, nz, diff);
    }
    static __device__ __forceinline__ void counts(uint32_t w, uint32_t& np1, uint32_t& nm1, uint32_t& n0)
    {
        cell_counts(w, np1, nm1, n0);
    }
    // neighbour word of cells i - 1 (even) / i + 1 (odd)
    static __device__ __forceinline__ uint32_t left(uint32_t w, uint32_t prev) { return funnel(w, prev, 28); }
    static __device__ __forceinline__ uint32_t right(uint32_t next, uint32_t w) { return funnel(next, w, 4); }
    static __device__ __forceinline__ int spin(const uint32_t* __restrict__ row, uint32_t i)
    {
        return (int)((row[i >> 3] >> (4 * (i & 7))) & 0xFu) - 1;
    }
};

template <>
struct Cell<1> {
    static constexpr int kPerWord = 32;
    static constexpr int kVecShift = 8;
    static constexpr int kWordShift = 6;
    static __device__ __forceinline__ void pair(uint32_t a, uint32_t b, uint32_t& nz, uint32_t& diff)
    {
        nz += 32;
        diff = bcnt_acc(a ^ b, diff);
    }
    // -1 cells: what the +1 cells leave (taken at the end of the pass)
    static __device__ __forceinline__ void counts(uint32_t w, uint32_t& np1, uint32_t&, uint32_t&)
    {
        np1 = bcnt_acc(w, np1);
    }
    static __device__ __forceinline__ uint32_t left(uint32_t w, uint32_t prev) { return funnel(w, prev, 31); }
    static __device__ __forceinline__ uint32_t right(uint32_t next, uint32_t w) { return funnel(next, w, 1); }
    static __device__ __forceinline__ int spin(const uint32_t* __restrict__ row, uint32_t i)
    {
        return ((row[i >> 5] >> (i & 31)) & 1u) ? 1 : -1;
    }
};

// Sum v[0..N) over the workgroup (wave sums, then across the waves in LDS)
// and add the totals to out[0..N): one atomic per value per workgroup, so
// the device-wide atomics on a handful of addresses stay few.
template <int N>
__device__ __forceinline__ void block_add(const int64_t (&v)[N], int64_t* __restrict__ out, int64_t (*lds)[N])
{
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int64_t s = wave_sum(v[i]);
        if ((threadIdx.x & 63) == 0) lds[wave][i] = s;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        int64_t tot = 0;
        for (int w = 0; w < nwaves; ++w) tot += lds[w][i];
        if (tot != 0) atomicAdd((unsigned long long*)&out[i], (unsigned long long)tot);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// B, M, Q, counts.  One thread per 16-byte column of plane 0, walking a
// band of rows with plane 1's rows y - 1, y, y + 1 in registers.
// ---------------------------------------------------------------------------
// Histogram of t = sigma h + 4 (0..8) over the cells of word o, whose four
// neighbour words are a, b (vertical), c (same row) and d (horizontal).
// 4-bit cells: the neighbour sum S = sum n = h + 4 fits a nibble, and
// t = 4 for sigma = 0, S for sigma = +1, 8 - S for sigma = -1.
__device__ __forceinline__ void sd_add4(uint32_t o, uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&hist)[9])
{
    const uint32_t S = a + b + c + d;
    const uint32_t e2 = (o >> 1) & 0x11111111u, e0 = ~(o | (o >> 1)) & 0x11111111u;
    const uint32_t m2 = shl_opaque<4>(e2) - e2;                    // 0xF where sigma = +1
    const uint32_t m0 = shl_opaque<4>(e0) - e0;                    // 0xF where sigma = -1
    const uint32_t t = (S & m2) | ((0x88888888u - S) & m0) | (0x44444444u & ~(m0 | m2));
    const uint32_t b0 = t & 0x11111111u, b1 = (t >> 1) & 0x11111111u;
    const uint32_t b2 = (t >> 2) & 0x11111111u, b3 = (t >> 3) & 0x11111111u;
    const uint32_t n0 = b0 ^ 0x11111111u, n1 = b1 ^ 0x11111111u, n2 = b2 ^ 0x11111111u, n3 = b3 ^ 0x11111111u;
    const uint32_t lo[4] = {n0 & n1, b0 & n1, n0 & b1, b0 & b1};
    const uint32_t hi0 = n2 & n3, hi1 = b2 & n3;
#pragma unroll
    for (int v = 0; v < 8; ++v) hist[v] = bcnt_acc(lo[v & 3] & (v < 4 ? hi0 : hi1), hist[v]);
    hist[8] = bcnt_acc(b3, hist[8]);
}

// 1-bit cells: t = 2 (aligned neighbours), from the four words of
// differences d_j = neighbour ^ own.
__device__ __forceinline__ void sd_add1(uint32_t o, uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t (&hist)[9])
{
    const uint32_t d0 = a ^ o, d1 = b ^ o, d2 = c ^ o, d3 = d ^ o;
    const uint32_t t1 = d0 ^ d1, t2 = d2 ^ d3;
    const uint32_t all_eq = ~(d0 | d1 | d2 | d3);                    // 4 aligned: t = 8
    const uint32_t all_ne = d0 & d1 & d2 & d3;                       // 0 aligned: t = 0
    const uint32_t one_ne = (t1 ^ t2) & ~((d0 & d1) | (d2 & d3));    // 3 aligned: t = 6
    const uint32_t one_eq = (t1 ^ t2) & (d0 | d1) & (d2 | d3);       // 1 aligned: t = 2
    hist[8] = bcnt_acc(all_eq, hist[8]);
    hist[0] = bcnt_acc(all_ne, hist[0]);
    hist[6] = bcnt_acc(one_ne, hist[6]);
    hist[2] = bcnt_acc(one_eq, hist[2]);
    // two aligned (t = 4): the rest of the cells, at the end of the pass
}

// 4-bit Ising cells (n in {0, 2}): per nibble S = 2 d, d the number of
// neighbours of the opposite sign, 0..4 (each xor nibble is 0 or 2, their
// sum at most 8), so bits 1, 2, 3 of the nibble are bits 0, 1, 2 of d.
// With n_k the number of cells with d = k, adds to
//   e[0] the set bits of S:            n_1 + n_2 + 2 n_3 + n_4,
//   e[1] those at nibble bit 1:        n_1 + n_3,
//   e[2] bits 1 and 2 both set:        n_3,
//   e[3] those at nibble bit 3:        n_4,
// from which the end of the pass takes n_1 .. n_4; n_0 is the rest of the
// cells, and the bond sum follows from the histogram.
__device__ __forceinline__ void sd_add_ising4(uint32_t o, uint32_t a, uint32_t b, uint32_t c, uint32_t d,
                                              uint32_t (&e)[4])
{
    const uint32_t S = xad(d, o, xad(c, o, xad(b, o, a ^ o)));
    e[0] = bcnt_acc(S, e[0]);
    e[1] = bcnt_acc(S & 0x22222222u, e[1]);
    e[2] = bcnt_acc(S & (S << 1) & 0x44444444u, e[2]);
    e[3] = bcnt_acc(S & 0x88888888u, e[3]);
}

// v of lane i + 1 (from_right) or lane i - 1 (from_left) of the wave, by a
// DPP wave shift; the lane at the end without a neighbour gets an
// unspecified value.
__device__ __forceinline__ uint32_t from_right(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, false);    // wave_shl:1
}
__device__ __forceinline__ uint32_t from_left(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, false);    // wave_shr:1
}

// One pass over both planes: B and M, Q and the value counts, and the
// Schwinger-Dyson histogram (section 4) of sigma h over every site.  A task
// is a column vector q of a band of rows; the thread keeps rows y - 1, y, y + 1 of both
// planes.  Colour-0 sites carry the bonds (each bond has one colour-0
// end); both colours add to the counts and the histogram.
// WAVE_ROWS: L / (cells per vector) is a multiple of 64, so the 64 lanes of
// a wave share their band and its row parity is a scalar.
template <int MODEL, bool WAVE_ROWS>
__global__ __launch_bounds__(256) void bmq_kernel(const uint32_t* __restrict__ p0, const uint32_t* __restrict__ p1,
                                                  uint32_t L, uint32_t rows, int64_t* __restrict__ acc)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    using C = Cell<CB>;
    __shared__ int64_t red[4][14];
    const uint32_t Q = L >> C::kVecShift, W = L >> C::kWordShift;
    const uint32_t tasks = Q * (L / rows);
    uint32_t nz = 0, diff = 0, np1 = 0, nm1 = 0, n0 = 0, cells = 0;
    uint32_t hist[9], e[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 9; ++k) hist[k] = 0;
    // workgroup ids go round-robin to the 8 XCDs: XCD x takes the x-th
    // eighth of the workgroups in order, so the tasks beside a workgroup's
    // (the rest of its bands, the bands above and below) run on the same
    // XCD at about the same time and the lines they share meet in its L2
    const uint32_t nb = gridDim.x;
    const uint32_t blk = (nb & 7u) == 0 ? (blockIdx.x & 7u) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    for (uint32_t g = blk * blockDim.x + threadIdx.x; g < tasks; g += nb * blockDim.x) {
        const uint32_t q = g % Q;
        uint32_t y0 = (g / Q) * rows;
        if (WAVE_ROWS) y0 = __builtin_amdgcn_readfirstlane(y0);
        const uint4* a4 = reinterpret_cast<const uint4*>(p0) + q;
        const uint4* b4 = reinterpret_cast<const uint4*>(p1) + q;
        const size_t yu = y0 == 0 ? L - 1 : y0 - 1;
        uint4 aup = a4[yu * Q], amid = a4[(size_t)y0 * Q];
        uint4 bup = b4[yu * Q], bmid = b4[(size_t)y0 * Q];
        const uint32_t hwl = (q == 0) ? W - 1 : 4 * q - 1;
        const uint32_t hwr = (4 * q + 4 == W) ? 0 : 4 * q + 4;
        // the words beside the vector are the neighbouring lanes' end words
        // (moved across by DPP), except at the ends of the wave or the row
        const uint32_t lane = threadIdx.x & 63u;
        const bool edge_l = lane == 0 || q == 0, edge_r = lane == 63 || q + 1 == Q;
        cells += 2 * C::kPerWord * 4 * rows;    // both planes, 4 words a row
        for (uint32_t r = 0; r < rows; ++r) {
            const uint32_t y = y0 + r;
            const size_t yd = (y + 1 == L) ? 0 : y + 1;
            const uint4 adn = a4[yd * Q], bdn = b4[yd * Q];
            const bool odd = (y & 1u) != 0;      // colour-0 sites of row y have x = 2 i + (y & 1)
            // colour 0 looks right (i + 1) on odd rows, colour 1 on even rows
            uint32_t bhalo = odd ? from_right(bmid.x) : from_left(bmid.w);
            uint32_t ahalo = odd ? from_left(amid.w) : from_right(amid.x);
            if (odd ? edge_r : edge_l) bhalo = p1[(size_t)y * W + (odd ? hwr : hwl)];
            if (odd ? edge_l : edge_r) ahalo = p0[(size_t)y * W + (odd ? hwl : hwr)];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const uint32_t wb = pick(bmid, d), wa = pick(amid, d);
                const uint32_t hb = odd ? C::right(d < 3 ? pick(bmid, d + 1) : bhalo, wb)
                                        : C::left(wb, d > 0 ? pick(bmid, d - 1) : bhalo);
                const uint32_t ha = odd ? C::left(wa, d > 0 ? pick(amid, d - 1) : ahalo)
                                        : C::right(d < 3 ? pick(amid, d + 1) : ahalo, wa);
                C::counts(wa, np1, nm1, n0);
                C::counts(wb, np1, nm1, n0);
                if (MODEL == 0) {
                    sd_add_ising4(wa, pick(bup, d), pick(bdn, d), wb, hb, e);
                    sd_add_ising4(wb, pick(aup, d), pick(adn, d), wa, ha, e);
                    continue;
                }
                C::pair(wa, pick(bup, d), nz, diff);
                C::pair(wa, pick(bdn, d), nz, diff);
                C::pair(wa, wb, nz, diff);
                C::pair(wa, hb, nz, diff);
                if (CB == 4) {
                    sd_add4(wa, pick(bup, d), pick(bdn, d), wb, hb, hist);
                    sd_add4(wb, pick(aup, d), pick(adn, d), wa, ha, hist);
                } else {
                    sd_add1(wa, pick(bup, d), pick(bdn, d), wb, hb, hist);
                    sd_add1(wb, pick(aup, d), pick(adn, d), wa, ha, hist);
                }
            }
            aup = amid;
            amid = adn;
            bup = bmid;
            bmid = bdn;
        }
    }
    int64_t bonds = (int64_t)nz - 2 * (int64_t)diff;
    if (MODEL == 0) {
        // n_1 .. n_4 from the sums of sd_add_ising4 (t = 8 - 2 d); the
        // thread's cells were 16 per word pair, the rest of the histogram
        // has d = 0; each bond is seen from both ends, so the bond sum is
        // 2 (cells) - sum of d over all cells
        hist[2] = e[2];
        hist[0] = e[3];
        hist[6] = e[1] - e[2];
        hist[4] = e[0] - e[1] - e[2] - e[3];
        hist[8] = cells - hist[6] - hist[4] - hist[2] - hist[0];
        const uint32_t dsum = hist[6] + 2 * hist[4] + 3 * hist[2] + 4 * hist[0];
        bonds = (int32_t)(2 * cells - dsum);    // (a thread's share may be negative)
    }
    if (MODEL == 2) {
        // 1-bit cells are all +1 or -1; t = 4 is what the other bins leave
        nm1 = cells - np1;
        hist[4] = cells - hist[0] - hist[2] - hist[6] - hist[8];
    }
    // acc: [0] B, [1] M, [2] #(+1), [3] #(-1), [4] #(0), [5 + k] #(sigma h = k - 4);
    // invalid cells are what the three counts leave of L^2 (done on the host)
    int64_t v[14] = {bonds, (int64_t)np1 - (int64_t)nm1, (int64_t)np1, (int64_t)nm1, (int64_t)n0};
#pragma unroll
    for (int k = 0; k < 9; ++k) v[5 + k] = (int64_t)hist[k];
    block_add<14>(v, acc, red);
}

// ---------------------------------------------------------------------------
// Correlations, every source, arbitrary r (full mode beyond r = 32): partners read
// from global memory.  One thread per (plane, band of rows, column), a
// chunk of up to kRChunk distances per grid row.
// ---------------------------------------------------------------------------
constexpr int kRChunk = 16;

// Word of the cells i + m .. (one word's worth, periodic in the row of W
// words), where cell i is cell 0 of word wd; wd + m / cells-per-word < 2 W.
template <int CB>
__device__ __forceinline__ uint32_t shifted_word(const uint32_t* __restrict__ row, uint32_t W, uint32_t wd, uint32_t m)
{
    const uint32_t mb = m * CB;
    const uint32_t w0 = wrap(wd + (mb >> 5), W);
    const uint32_t w1 = wrap(w0 + 1, W);
    return funnel(row[w1], row[w0], mb & 31);
}

template <int CB>
__global__ __launch_bounds__(256) void corr_all_kernel(const uint32_t* __restrict__ planes, uint32_t L, uint32_t rows,
                                                       const int32_t* __restrict__ rlist, int nr,
                                                       int64_t* __restrict__ Cx, int64_t* __restrict__ Cy)
{
    using Cl = Cell<CB>;
    const uint32_t Q = L >> Cl::kVecShift, W = L >> Cl::kWordShift;
    const int j0 = blockIdx.y * kRChunk;
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t q = g % Q;
    const uint32_t rest = g / Q;
    const uint32_t nbands = L / rows;
    const uint32_t c = rest / nbands;
    const uint32_t band = rest - c * nbands;
    const size_t plane_words = (size_t)L * W;
    uint32_t xn[kRChunk], xd[kRChunk], yn[kRChunk], yd[kRChunk];
#pragma unroll
    for (int j = 0; j < kRChunk; ++j) xn[j] = xd[j] = yn[j] = yd[j] = 0;
    if (c < 2) {
        const uint32_t* own = planes + (c ? plane_words : 0);
        for (uint32_t rr = 0; rr < rows; ++rr) {
            const uint32_t y = band * rows + rr;
            const uint4 v = reinterpret_cast<const uint4*>(own)[(size_t)y * Q + q];
            const uint32_t par = (y + c) & 1u;
#pragma unroll
            for (int j = 0; j < kRChunk; ++j) {
                if (j0 + j < nr) {
                    const uint32_t r = (uint32_t)rlist[j0 + j];
                    const uint32_t pc = c ^ (r & 1u);
                    const uint32_t* pl = planes + (pc ? plane_words : 0);
                    const uint32_t yr = wrap(y + r, L);
                    const uint4 py = reinterpret_cast<const uint4*>(pl)[(size_t)yr * Q + q];
                    const uint32_t m = (r & 1u) ? ((r - 1) >> 1) + par : (r >> 1);
                    const uint32_t* prow = pl + (size_t)y * W;
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const uint32_t o = pick(v, d);
                        Cl::pair(o, pick(py, d), yn[j], yd[j]);
                        Cl::pair(o, shifted_word<CB>(prow, W, 4 * q + d, m), xn[j], xd[j]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kRChunk; ++j) {
        const int64_t sx = wave_sum((int64_t)xn[j] - 2 * (int64_t)xd[j]);
        const int64_t sy = wave_sum((int64_t)yn[j] - 2 * (int64_t)yd[j]);
        if ((threadIdx.x & 63) == 0 && j0 + j < nr) {
            atomicAdd((unsigned long long*)&Cx[j0 + j], (unsigned long long)sx);
            atomicAdd((unsigned long long*)&Cy[j0 + j], (unsigned long long)sy);
        }
    }
}

// ---------------------------------------------------------------------------
// Correlations, sampled sources (x = y = 0 mod 16), as bits.
//
// T bits (layout in internal.h): for every row y, bit j of word k is
// [s(16 a, y) = +1] with a = 32 k + j, and for Blume-Capel a second plane
// holds [s(16 a, y) != 0]; below L = 512 the NS = L / 16 bits of a row repeat
// to fill its one word (NS divides 32), so a rotation by m of the word is a
// shift by m mod NS.  The site (16 a, y) has colour y & 1 and in-plane index
// 8 a.
//
// A sum of s s' over the pairs of two such words is, with the mask z of the
// pairs that count (both nonzero, and inside the row), popc(z) - 2
// popc(z & (a ^ b)): a product is +1 for equal signs and -1 otherwise.
// ---------------------------------------------------------------------------
template <int MODEL>
__device__ __forceinline__ int sampled_pairs(uint32_t s, uint32_t sz, uint32_t p, uint32_t pz, uint32_t valid,
                                             bool full)
{
    if (MODEL == 1) {
        const uint32_t z = sz & pz & valid;
        return (int)popc(z) - 2 * (int)popc(z & (s ^ p));
    }
    if (full) return 32 - 2 * (int)popc(s ^ p);
    return (int)popc(valid) - 2 * (int)popc(valid & (s ^ p));
}

// T bits below L = 512, where the measurement pass does not write them:
// thread per row, whose NS bits fill one word.
template <int MODEL>
__global__ __launch_bounds__(256) void tbits_kernel(const uint32_t* __restrict__ planes, uint32_t L,
                                                    uint32_t* __restrict__ tb)
{
    using C = Cell<MODEL == 2 ? 1 : 4>;
    const uint32_t W = L >> C::kWordShift, NS = L >> 4;
    const size_t plane_words = (size_t)L * W;
    const uint32_t y = blockIdx.x * blockDim.x + threadIdx.x;
    if (y >= L) return;
    const uint32_t* row = planes + (y & 1u) * plane_words + (size_t)y * W;
    uint32_t sb = 0, zb = 0;
    for (uint32_t j = 0; j < 32; ++j) {
        const int s = C::spin(row, 8u * (j % NS));
        sb |= (s > 0 ? 1u : 0u) << j;
        zb |= (s != 0 ? 1u : 0u) << j;
    }
    const uint32_t at = (y & 15u) * NS + (y >> 4);
    tb[at] = sb;
    if (MODEL == 1) tb[L + at] = zb;
}

// Along x, one sampled row y = 16 b at a time (persistent over rows).  The
// row's cells go into LDS as residue rows of bits: R_rho bit a is the cell
// (16 a + rho, y).  R_0 holds the sources, and the partners of distance
// r = 16 m + rho are R_rho shifted by m: per word of 32 sources one funnel
// shift, one xor and the bit counts.  LDS holds R_0 and the residues rho0 ..
// rho0 + G - 1 (the host runs 16 / G passes when a row of all 16 residues
// does not fit), each residue row twice in a row, so the partner words
// w + m / 32 and the next need no wrap, and two words of padding after each
// row, so the rows of different residues start in different LDS banks.
// Thread k owns distance k of the launch (the host gives a launch at most
// one distance per thread): it walks every word of the row, reading the
// source words as broadcast 16-byte loads, and keeps its sum in a register
// over all the workgroup's rows; one atomic per distance and workgroup at
// the end.  Workgroups of 512 threads, several per CU, so one loads its next
// row while another works on its own.  For 4-bit Ising lattices from L = 512
// on (rb set) the residue rows come ready from the measurement pass, and the
// row's 4-bit cells are not read at all.  (Lanes over the words and a wave's
// distances in registers, which frees the LDS reads of bank conflicts, took
// 193 us at L = 2^17 where this takes 162: a third of the time is building
// the rows, and 64 sums to reduce per wave cost what the conflicts did.)
//
// Building the residue rows (L >= 512): a 4-bit word w of plane c holds the
// cells x = 16 w + 2 j + c, j = 0 .. 7, i.e. bit w of residues 2 j + c, so a
// wave's 64 words give 64 bits of each of its residues by one ballot per j.
// A 1-bit word w of plane c holds x = 64 w + 2 k + c: bit k belongs to
// residue 2 (k & 7) + c at position 4 w + (k >> 3), four bits per residue,
// gathered per lane and merged over 8 lanes.
constexpr uint32_t kSxU = 4;        // row loads in flight per thread
constexpr int kSxThreads = 512;     // threads of a workgroup, and distances of a launch

__device__ __forceinline__ int sx_row(uint32_t rho, uint32_t rho0, uint32_t G)
{
    return rho - rho0 < G ? (int)(1 + rho - rho0) : -1;
}

template <int MODEL>
__global__ __launch_bounds__(kSxThreads) void corr_sxb_kernel(const uint32_t* __restrict__ planes,
                                                      const uint32_t* __restrict__ rb, uint32_t L,
                                                       const int32_t* __restrict__ rlist, int nr, uint32_t rho0,
                                                       uint32_t G, int64_t* __restrict__ Cx)
{
    constexpr int NB = MODEL == 1 ? 2 : 1;
    using C = Cell<MODEL == 2 ? 1 : 4>;
    extern __shared__ int sxb_lds[];
    uint32_t* R = reinterpret_cast<uint32_t*>(sxb_lds);   // [(1 + G) rows][NB][2 NSW], + 2 words a row
    const uint32_t W = L >> C::kWordShift, NS = L >> 4;
    const uint32_t NSW = L >= 512 ? L >> 9 : 1u;
    const uint32_t PO = 2 * NSW;                          // bit plane offset within a row
    const uint32_t rowstride = NB * PO + 2;
    const bool full = L >= 512;
    // Ising rows without invalid bits: a word's sum is 32 - 2 (differing bits)
    const bool diff_only = MODEL != 1 && full;
    const uint32_t valid = full ? 0xFFFFFFFFu : (NS >= 32 ? 0xFFFFFFFFu : ((1u << NS) - 1u));
    const size_t plane_words = (size_t)L * W;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nwaves = blockDim.x >> 6;
    // this thread's distance: r = 16 m + rho, the partners R_rho shifted by m
    const int k = threadIdx.x;
    const uint32_t r = k < nr ? (uint32_t)rlist[k] : 0u;
    const int rr = k < nr ? sx_row(r & 15u, rho0, G) : -1;     // -1: none, or another pass's residue
    const uint32_t m = r >> 4, sh = m & 31u;
    const uint32_t poff = (rr < 0 ? 0u : (uint32_t)rr * rowstride) + (m >> 5);
    uint32_t acc = 0;
    uint32_t rows_done = 0;
    for (uint32_t b = blockIdx.x; b < NS; b += gridDim.x) {
        const uint32_t y = 16 * b;
        ++rows_done;
        __syncthreads();
        if (MODEL == 0 && rb != nullptr) {
            // the residue rows the measurement pass wrote, 16 of them word by
            // word: row 0 takes the sources (residue 0), rows 1 .. G the
            // residues rho0 .., each stored twice; kSxU loads in flight per thread
            const uint32_t* src = rb + (size_t)b * NSW * 16;
            const uint32_t total = NSW * 16;
            for (uint32_t base = threadIdx.x; base < total; base += kSxU * blockDim.x) {
                uint32_t v[kSxU];
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t t = base + u * blockDim.x;
                    v[u] = t < total ? src[t] : 0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t t = base + u * blockDim.x;
                    if (t >= total) break;
                    const uint32_t rho = t & 15u, w = t >> 4, slot = rho - rho0;
                    if (rho == 0) R[w] = v[u];
                    if (slot < G) {
                        uint32_t* row = R + (1 + slot) * rowstride + w;
                        row[0] = v[u];
                        row[NSW] = v[u];
                    }
                }
            }
        } else if (L < 512) {
            // one word per residue row, its NS bits repeated
            for (uint32_t t = threadIdx.x; t < (1 + G) * NB; t += blockDim.x) {
                const uint32_t rr = t / NB, plane = t - rr * NB;
                const uint32_t rho = rr == 0 ? 0u : rho0 + rr - 1;
                const uint32_t c = rho & 1u;                     // (x + y) & 1 with y even
                const uint32_t* row = planes + c * plane_words + (size_t)y * W;
                uint32_t v = 0;
                for (uint32_t j = 0; j < 32; ++j) {
                    const int s = C::spin(row, (16u * (j % NS) + rho) >> 1);
                    v |= ((plane == 0 ? s > 0 : s != 0) ? 1u : 0u) << j;
                }
                R[rr * rowstride + plane * PO] = v;
            }
        } else if (C::kPerWord == 8) {
            // a wave takes 64 consecutive words of the row at a time (2 W of
            // them, both planes; W is a multiple of 32, so a group of 64 is
            // whole): the bookkeeping is per wave.  The loads of kSxU groups
            // are issued together, so a wave waits for memory once per kSxU
            // groups rather than once per group.
            const uint32_t step = 64u * (uint32_t)nwaves;
            for (uint32_t base = __builtin_amdgcn_readfirstlane(64u * (uint32_t)wave); base < 2 * W;
                 base += kSxU * step) {
                uint32_t words[kSxU];
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t idx = base + u * step + (uint32_t)lane;
                    const uint32_t c = idx >= W ? 1u : 0u;
                    words[u] = idx < 2 * W ? planes[c * plane_words + (size_t)y * W + (idx - c * W)] : 0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t idx0 = base + u * step;
                    if (idx0 >= 2 * W) break;
                    const uint32_t word = words[u];
                    // lanes 0..31 and 32..63 cover 32 words each, of one plane each
                    const uint32_t c_lo = idx0 >= W ? 1u : 0u, c_hi = idx0 + 32 >= W ? 1u : 0u;
                    const uint32_t k_lo = (idx0 - c_lo * W) >> 5, k_hi = (idx0 + 32 - c_hi * W) >> 5;
                    uint64_t ms[8], mz[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        ms[j] = __ballot((word >> (4 * j + 1)) & 1u);
                        mz[j] = NB == 2 ? __ballot(((~word) >> (4 * j)) & 1u) : 0u;
                    }
                    if (c_lo == c_hi) {
                        // L >= 1024: the two halves are words k_lo, k_lo + 1 (k_lo
                        // even) of one residue row, 8-byte aligned in LDS
                        if (lane == 0) {
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                const uint32_t t = 2u * j + c_lo - rho0;       // the residue's slot - 1
                                if (t < G) {
                                    uint32_t* dst = R + (1 + t) * rowstride + k_lo;
                                    *reinterpret_cast<uint2*>(dst) = make_uint2((uint32_t)ms[j], (uint32_t)(ms[j] >> 32));
                                    if (NB == 2)
                                        *reinterpret_cast<uint2*>(dst + PO) =
                                            make_uint2((uint32_t)mz[j], (uint32_t)(mz[j] >> 32));
                                }
                            }
                            if (c_lo == 0) {                                   // residue 0: the sources
                                *reinterpret_cast<uint2*>(R + k_lo) = make_uint2((uint32_t)ms[0], (uint32_t)(ms[0] >> 32));
                                if (NB == 2)
                                    *reinterpret_cast<uint2*>(R + PO + k_lo) =
                                        make_uint2((uint32_t)mz[0], (uint32_t)(mz[0] >> 32));
                            }
                        }
                        continue;
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        if (lane == 0) {
                            const uint32_t rl_lo = 2 * j + c_lo, rl_hi = 2 * j + c_hi;
                            const int r_lo = sx_row(rl_lo, rho0, G), r_hi = sx_row(rl_hi, rho0, G);
                            if (r_lo >= 0) {
                                R[r_lo * rowstride + k_lo] = (uint32_t)ms[j];
                                if (NB == 2) R[r_lo * rowstride + PO + k_lo] = (uint32_t)mz[j];
                            }
                            if (r_hi >= 0) {
                                R[r_hi * rowstride + k_hi] = (uint32_t)(ms[j] >> 32);
                                if (NB == 2) R[r_hi * rowstride + PO + k_hi] = (uint32_t)(mz[j] >> 32);
                            }
                            if (rl_lo == 0) {                            // the sources
                                R[k_lo] = (uint32_t)ms[j];
                                if (NB == 2) R[PO + k_lo] = (uint32_t)mz[j];
                            }
                            if (rl_hi == 0) {
                                R[k_hi] = (uint32_t)(ms[j] >> 32);
                                if (NB == 2) R[PO + k_hi] = (uint32_t)(mz[j] >> 32);
                            }
                        }
                    }
                }
            }
        } else {
            // as above, the loads of kSxU words per thread issued together
            for (uint32_t base = threadIdx.x; base < 2 * W; base += kSxU * blockDim.x) {
                uint32_t words[kSxU];
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t idx = base + u * blockDim.x;
                    const uint32_t c = idx >= W ? 1u : 0u;
                    words[u] = idx < 2 * W ? planes[c * plane_words + (size_t)y * W + (idx - c * W)] : 0u;
                }
#pragma unroll
                for (uint32_t u = 0; u < kSxU; ++u) {
                    const uint32_t idx = base + u * blockDim.x;
                    if (idx >= 2 * W) break;
                    const uint32_t c = idx >= W ? 1u : 0u;
                    const uint32_t w = idx - c * W;
                    const uint32_t word = words[u];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const uint32_t x = (word >> j) & 0x01010101u;     // bits j, j + 8, j + 16, j + 24
                        const uint32_t nib = (x | (x >> 7) | (x >> 14) | (x >> 21)) & 0xFu;
                        uint32_t v = nib << (4u * (w & 7u));
                        v |= __shfl_xor(v, 1);
                        v |= __shfl_xor(v, 2);
                        v |= __shfl_xor(v, 4);
                        if ((w & 7u) == 0) {
                            const uint32_t rho = 2 * j + c;
                            const int rr = sx_row(rho, rho0, G);
                            if (rr >= 0) R[rr * rowstride + (w >> 3)] = v;
                            if (rho == 0) R[w >> 3] = v;
                        }
                    }
                }
            }
        }
        __syncthreads();
        // the second copy of each residue row (the packed rows come with it)
        for (uint32_t t = threadIdx.x; !(MODEL == 0 && rb != nullptr) && t < G * NB * NSW; t += blockDim.x) {
            const uint32_t rr = 1 + t / (NB * NSW), rest = t % (NB * NSW);
            const uint32_t pl = rest / NSW, w = rest - pl * NSW;
            uint32_t* row = R + rr * rowstride + pl * PO;
            row[NSW + w] = row[w];
        }
        __syncthreads();
        if (rr >= 0) {
            const uint32_t* P = R + poff;
            if (diff_only && (NSW & 3u) == 0) {
                for (uint32_t w = 0; w < NSW; w += 4) {
                    const uint4 s4 = *reinterpret_cast<const uint4*>(R + w);
                    const uint32_t p0 = P[w], p1 = P[w + 1], p2 = P[w + 2], p3 = P[w + 3], p4 = P[w + 4];
                    acc = bcnt_acc(s4.x ^ funnel(p1, p0, sh), acc);
                    acc = bcnt_acc(s4.y ^ funnel(p2, p1, sh), acc);
                    acc = bcnt_acc(s4.z ^ funnel(p3, p2, sh), acc);
                    acc = bcnt_acc(s4.w ^ funnel(p4, p3, sh), acc);
                }
            } else {
                for (uint32_t w = 0; w < NSW; ++w) {
                    const uint32_t p = funnel(P[w + 1], P[w], sh);
                    if (diff_only) {
                        acc = bcnt_acc(R[w] ^ p, acc);
                    } else {
                        uint32_t sz = 0, pz = 0;
                        if (NB == 2) {
                            sz = R[PO + w];
                            pz = funnel(P[PO + w + 1], P[PO + w], sh);
                        }
                        acc += (uint32_t)sampled_pairs<MODEL>(R[w], sz, p, pz, valid, full);
                    }
                }
            }
        }
    }
    // Ising from L = 512 on: the sum counts differing bits (32 pairs a word)
    if (rr >= 0) {
        const int64_t v = diff_only ? 32 * (int64_t)NSW * rows_done - 2 * (int64_t)acc : (int64_t)(int32_t)acc;
        if (v != 0) atomicAdd((unsigned long long*)&Cx[k], (unsigned long long)v);
    }
}

// Along y: S_y(r) = sum over the sampled rows b and words k of the pairs of
// T row 16 b and T row 16 b + r (mod L).  With r = 16 q + rho the partner rows
// are those of residue class rho from b + q on, which the T bits hold one
// after the other for each word.  A workgroup takes one word k and one class:
// its NS words go to LDS (the first half twice, so that b + q needs no wrap:
// 48 KiB at L = 2^17), and a thread walks the source words b, kYGroup
// distances of the class at a time, one LDS read, xor and bit count each,
// neighbouring lanes reading neighbouring words.  Each word of the T bits is
// read once as a partner, however many distances there are, and the kernel is
// bound by the LDS reads.  4-bit Ising L = 2^17, 480 distances: 0.23 ms; with
// the T bits row by row, partners read from the last-level cache, 0.43.
// STAGED false: classes that do not fit LDS are read from memory (L = 2^20,
// and Blume-Capel at L = 2^19).
// DIFF (Ising from L = 512 on): no word has invalid bits, so the sum is 32 per
// word minus twice the count of differing bits, which is all the loop counts.
constexpr int kYGroup = 8;
constexpr int kYUnroll = 4;
constexpr int kYThreads = 256;

// The source words b, b + kYThreads, .. (U of them) against kYGroup partners
// at offsets q.
template <int NB, bool STAGED, bool DIFF, int U>
__device__ __forceinline__ void sy_rows(const uint32_t* src, size_t zoff, const uint32_t* part, size_t part_z,
                                        uint32_t NS, uint32_t valid, uint32_t b, const uint32_t (&q)[kYGroup],
                                        uint32_t (&acc)[kYGroup])
{
    uint32_t s[U], sz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        s[u] = src[b + u * kYThreads];
        sz[u] = NB == 2 ? src[zoff + b + u * kYThreads] : 0u;
    }
#pragma unroll
    for (int j = 0; j < kYGroup; ++j) {
        const uint32_t* p = part + b + q[j];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t* at = STAGED ? p + u * kYThreads : part + ((b + q[j] + u * kYThreads) & (NS - 1));
            if (DIFF)
                acc[j] = bcnt_acc(s[u] ^ *at, acc[j]);
            else
                acc[j] += (uint32_t)sampled_pairs<NB == 2 ? 1 : 0>(s[u], sz[u], *at, NB == 2 ? at[part_z] : 0u, valid,
                                                                   false);
        }
    }
}

template <int NB, bool STAGED, bool DIFF>
__global__ __launch_bounds__(kYThreads) void corr_sy_kernel(const uint32_t* __restrict__ tb, uint32_t L,
                                                            const int32_t* __restrict__ rlist, int nr,
                                                            int64_t* __restrict__ Cy)
{
    extern __shared__ uint32_t cls[];                     // STAGED: [NB][NS + NS / 2]
    __shared__ int s_index[kYGroup + kYThreads], s_shift[kYGroup + kYThreads];
    __shared__ int s_n;
    __shared__ uint32_t red[kYThreads / 64][kYGroup];
    const uint32_t NS = L >> 4;
    const uint32_t NSW = L >= 512 ? L >> 9 : 1u;
    const uint32_t valid = NS >= 32 ? 0xFFFFFFFFu : ((1u << NS) - 1u);
    const uint32_t rho = blockIdx.x & 15u, k = blockIdx.x >> 4;
    const uint32_t* src = tb + (size_t)k * L;             // class 0: the sources
    const uint32_t* part = src + rho * NS;
    const size_t zoff = (size_t)L * NSW;                  // plane 1 (Blume-Capel nonzero bits)
    const uint32_t len = NS + NS / 2;                     // r <= L / 2: q <= NS / 2
    if (threadIdx.x == 0) s_n = 0;
    if (STAGED)
        for (uint32_t i = threadIdx.x; i < len; i += kYThreads) {
            cls[i] = part[i & (NS - 1)];
            if (NB == 2) cls[len + i] = part[zoff + (i & (NS - 1))];
        }
    __syncthreads();
    for (int base = 0;;) {
        // the next distances of the class: at least kYGroup of them, or the last
        int n = s_n;
        while (n < kYGroup && base < nr) {
            const int i = base + (int)threadIdx.x;
            const uint32_t r = i < nr ? (uint32_t)rlist[i] : 0u;
            __syncthreads();                              // every thread has read s_n
            if (i < nr && (r & 15u) == rho) {
                const int at = atomicAdd(&s_n, 1);
                s_index[at] = i;
                s_shift[at] = (int)(r >> 4);
            }
            base += kYThreads;
            __syncthreads();
            n = s_n;
        }
        if (n == 0) break;
        // (past the last distance: the sources themselves, and no sum)
        const int kn = min(n, kYGroup);
        uint32_t q[kYGroup], acc[kYGroup];
#pragma unroll
        for (int j = 0; j < kYGroup; ++j) {
            q[j] = (uint32_t)__builtin_amdgcn_readfirstlane(j < kn ? s_shift[j] : 0);
            acc[j] = 0;
        }
        const uint32_t* from = STAGED ? cls : part;
        const size_t from_z = STAGED ? len : zoff;
        if (NS % (kYThreads * kYUnroll) == 0) {
            for (uint32_t b = threadIdx.x; b < NS; b += kYThreads * kYUnroll)
                sy_rows<NB, STAGED, DIFF, kYUnroll>(src, zoff, from, from_z, NS, valid, b, q, acc);
        } else {
            for (uint32_t b = threadIdx.x; b < NS; b += kYThreads)
                sy_rows<NB, STAGED, DIFF, 1>(src, zoff, from, from_z, NS, valid, b, q, acc);
        }
#pragma unroll
        for (int j = 0; j < kYGroup; ++j) {
            const int v = wave_sum_i32((int)acc[j]);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = (uint32_t)v;
        }
        __syncthreads();
        if ((int)threadIdx.x < kn) {
            int64_t v = 0;
            for (int w = 0; w < kYThreads / 64; ++w) v += (int32_t)red[w][threadIdx.x];
            if (DIFF) v = 32 * (int64_t)NS - 2 * v;
            if (v != 0) atomicAdd((unsigned long long*)&Cy[s_index[threadIdx.x]], (unsigned long long)v);
        }
        // the distances that follow the group move up
        const bool rest = (int)threadIdx.x < n - kn;
        const int index = rest ? s_index[kn + threadIdx.x] : 0, shift = rest ? s_shift[kn + threadIdx.x] : 0;
        __syncthreads();
        if (rest) {
            s_index[threadIdx.x] = index;
            s_shift[threadIdx.x] = shift;
        }
        if (threadIdx.x == 0) s_n = n - kn;
        __syncthreads();
    }
}

int64_t pick_rows(int64_t L, int64_t want)
{
    int64_t rows = want;
    while (rows > 1 && (L % rows) != 0) rows >>= 1;
    return rows;
}

}  // namespace

hipError_t launch_begin(int64_t* acc, int64_t* Cx, int64_t* Cy, int nr, int32_t* rdev, const int32_t* host_r,
                        hipStream_t s)
{
    const dim3 grid((uint32_t)((std::max(nr, kAccSlots) + 255) / 256));
    hipLaunchKernelGGL(begin_kernel, grid, dim3(256), 0, s, acc, Cx, Cy, nr, rdev, host_r);
    return hipGetLastError();
}

hipError_t launch_finish(const int64_t* acc, const int64_t* Cx, const int64_t* Cy, int nr, int64_t* host, hipStream_t s)
{
    const dim3 grid((uint32_t)((std::max(nr, kAccSlots) + 255) / 256));
    hipLaunchKernelGGL(finish_kernel, grid, dim3(256), 0, s, acc, Cx, Cy, nr, host);
    return hipGetLastError();
}

// Optional band height of the B/M/Q pass: MCL_MEASURE_ROWS (2 to 64, read
// at every launch; the largest divisor of L up to it is taken).  Like the
// grid cap it changes the split of the work only; a test uses it to run the
// 64-row bands of large lattices at small L.
int64_t bmq_rows(const Geom& g)
{
    if (const char* e = std::getenv("MCL_MEASURE_ROWS")) {
        const long long v = std::atoll(e);
        if (v >= 2 && v <= 64) return pick_rows(g.L, v);
    }
    return pick_rows(g.L, g.Q * (g.L / 64) >= (int64_t(1) << 20) ? 64 : 32);
}

hipError_t launch_bmq(const Geom& g, int model, int64_t* acc, hipStream_t s)
{
    // one thread per task, bands of 64 rows while that leaves 2^20 tasks or
    // more (else 32).  The words beside a vector come from the neighbouring
    // lanes, so the lines a pass reads twice are the halo rows of its bands
    // and those at workgroup edges.  Measured at L = 2^17 (4-bit Ising),
    // bytes read against the lattice's: 1.50x with every halo word loaded
    // from memory, 1.12x with lane exchanges, 1.09x with the XCD-aware
    // workgroup order as well, 1.056x with 64-row bands (16 rows: 1.15x);
    // 2.06 - 2.09 ms each way once the halo loads were gone.
    const int64_t rows = bmq_rows(g);
    const int64_t threads = g.Q * (g.L / rows);
    const uint32_t grid = measure_grid_cap((uint32_t)((threads + 255) / 256));
    const uint32_t L = (uint32_t)g.L, R = (uint32_t)rows;
    const bool wave_rows = (g.Q & 63) == 0;
    if (model == 2) {
        if (wave_rows)
            hipLaunchKernelGGL((bmq_kernel<2, true>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
        else
            hipLaunchKernelGGL((bmq_kernel<2, false>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
    } else if (model == 1) {
        if (wave_rows)
            hipLaunchKernelGGL((bmq_kernel<1, true>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
        else
            hipLaunchKernelGGL((bmq_kernel<1, false>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
    } else {
        if (wave_rows)
            hipLaunchKernelGGL((bmq_kernel<0, true>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
        else
            hipLaunchKernelGGL((bmq_kernel<0, false>), dim3(grid), dim3(256), 0, s, g.plane(0), g.plane(1), L, R, acc);
    }
    return hipGetLastError();
}

hipError_t launch_tbits(const Geom& g, int model, uint32_t* tbits, hipStream_t s)
{
    if (g.L >= 512) return hipErrorInvalidValue;
    const dim3 grid((uint32_t)((g.L + 255) / 256));
    const uint32_t L = (uint32_t)g.L;
    if (model == 2) hipLaunchKernelGGL(tbits_kernel<2>, grid, dim3(256), 0, s, g.plane0, L, tbits);
    else if (model == 1) hipLaunchKernelGGL(tbits_kernel<1>, grid, dim3(256), 0, s, g.plane0, L, tbits);
    else hipLaunchKernelGGL(tbits_kernel<0>, grid, dim3(256), 0, s, g.plane0, L, tbits);
    return hipGetLastError();
}

bool bmq_fused()
{
    if (const char* e = std::getenv("MCL_MEASURE_FUSED")) return std::atoi(e) != 0;
    return true;
}

hipError_t launch_corr_all(const Geom& g, const int32_t* r_dev, int nr, int64_t* Cx, int64_t* Cy, hipStream_t s)
{
    if (nr <= 0) return hipSuccess;
    const int64_t rows = pick_rows(g.L, 16);
    const int64_t threads = 2 * g.Q * (g.L / rows);
    const uint32_t chunks = (uint32_t)((nr + kRChunk - 1) / kRChunk);
    const dim3 grid((uint32_t)((threads + 255) / 256), chunks);
    if (g.cb == 1)
        hipLaunchKernelGGL(corr_all_kernel<1>, grid, dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)rows, r_dev,
                           nr, Cx, Cy);
    else
        hipLaunchKernelGGL(corr_all_kernel<4>, grid, dim3(256), 0, s, g.plane0, (uint32_t)g.L, (uint32_t)rows, r_dev,
                           nr, Cx, Cy);
    return hipGetLastError();
}

namespace {

// LDS bytes the x-correlation kernel may use: 160 KiB, or less when the
// environment variable MCL_SX_LDS_BUDGET says so (a test uses it to run the
// multi-pass form at small L).
size_t sx_lds_budget()
{
    size_t budget = kLdsBytes;
    if (const char* e = std::getenv("MCL_SX_LDS_BUDGET")) {
        const long long v = std::atoll(e);
        if (v > 0 && (size_t)v < budget) budget = (size_t)v;
    }
    return budget;
}

template <int MODEL>
hipError_t corr_sampled_x(const Geom& g, const SampledArgs& a, hipStream_t s)
{
    const uint32_t L = (uint32_t)g.L, NS = L / 16;
    if ((L & (L - 1)) != 0 || L < 64) return hipErrorInvalidValue;   // the protocol's lattices only
    if (a.rbits && (MODEL != 0 || L < 512)) return hipErrorInvalidValue;
    constexpr int NB = MODEL == 1 ? 2 : 1;
    // along x: LDS holds the source row and G residue rows of bits, each
    // row stored twice and padded by two words; a launch takes one distance
    // per thread
    const size_t rowb = ((size_t)NB * 2 * tbits_words(L) + 2) * 4, budget = sx_lds_budget();
    const uint32_t gx = measure_grid_cap(std::min<uint32_t>(NS, 1024));
    uint32_t G = 16;
    while (G > 1 && rowb * (1 + G) > budget) G >>= 1;
    if (rowb * (1 + G) > budget) return hipErrorInvalidValue;
    const int max_r = kSxThreads;
    hipError_t e = hipSuccess;
    for (int j0 = 0; j0 < a.nr; j0 += max_r) {
        const int nr = std::min(max_r, a.nr - j0);
        const size_t lds = rowb * (1 + G);
        e = allow_lds(corr_sxb_kernel<MODEL>, lds, kLdsBytes);
        if (e != hipSuccess) return e;
        for (uint32_t rho0 = 0; rho0 < 16; rho0 += G) {
            hipLaunchKernelGGL((corr_sxb_kernel<MODEL>), dim3(gx), dim3(kSxThreads), lds, s, g.plane0, a.rbits, L, a.r + j0, nr, rho0,
                               G, a.Cx + j0);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

hipError_t corr_sampled_y(const Geom& g, int model, const SampledArgs& a, hipStream_t s)
{
    const uint32_t L = (uint32_t)g.L, NS = L / 16;
    if ((L & (L - 1)) != 0 || L < 64) return hipErrorInvalidValue;
    const size_t need = (model == 1 ? 2 : 1) * (size_t)(NS + NS / 2) * 4;
    constexpr size_t kMost = 152 * 1024;                  // with the kernel's own arrays, a workgroup's 160 KiB
    const bool staged = need <= kMost;
    const auto go = [&](auto kernel) {
        const hipError_t e = allow_lds(kernel, staged ? need : 0, kMost);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(16u * (uint32_t)tbits_words(L)), dim3(kYThreads), staged ? need : 0, s, a.tbits, L,
                           a.r, a.nr, a.Cy);
        return hipGetLastError();
    };
    if (model == 1) return staged ? go(corr_sy_kernel<2, true, false>) : go(corr_sy_kernel<2, false, false>);
    if (L < 512) return go(corr_sy_kernel<1, true, false>);
    return staged ? go(corr_sy_kernel<1, true, true>) : go(corr_sy_kernel<1, false, true>);
}

}  // namespace

hipError_t launch_corr_sampled_x(const Geom& g, int model, const SampledArgs& a, hipStream_t s)
{
    if (a.nr <= 0) return hipSuccess;
    return model == 2 ? corr_sampled_x<2>(g, a, s) : model == 1 ? corr_sampled_x<1>(g, a, s) : corr_sampled_x<0>(g, a, s);
}

hipError_t launch_corr_sampled_y(const Geom& g, int model, const SampledArgs& a, hipStream_t s)
{
    if (a.nr <= 0) return hipSuccess;
    return corr_sampled_y(g, model, a, s);
}

}  // namespace mcl
