// The measurement pass for gfx950: every-source correlations r = 0 .. 32
// along both axes, B, M, Q, the value counts and the Schwinger-Dyson
// histogram, and the bits of the sampled columns and rows, from one read of
// the lattice (sections 3.3 and 4).
//
// The correlations are contractions, and run on the matrix cores.  A 4-bit
// cell n = s + 1 read as an fp4 (E2M1) number is n / 2 exactly (0, 0.5, 1), so
// with P(r) the sum over all sources of (n / 2)(n' / 2),
//     C(r) = sum s s' = sum (n n' - n - n' + 1) = 4 P(r) - 2 sum n + L^2,
// the cells of a lattice row go into v_mfma_f32_16x16x128_f8f6f4 as they
// are, and the sums are exact: they are multiples of 1/4 below 2^22.
//
// U_p(y, i) is the site x = 2 i + p of row y: cell i of row y of plane
// (p + y) & 1.  In these terms neither parity nor colour enters a neighbour:
//   along y  U_p(y, i) meets U_p(y + r, i);
//   along x  U_p(y, i) meets U_p(y, i + m) at r = 2 m, U_0(y, i) meets
//            U_1(y, i + o) at r = 2 o + 1, U_1(y, i) meets U_0(y, i + o) at
//            r = 2 o - 1.
// Along y a 16x16 block product of rows [a, a + 16) and [b, b + 16) over 128
// cells gives all their pairs at r = b - a + j - i: three products per block
// of target rows cover r = 0 .. 32.  Along x the operands are 16 columns by
// 128 rows, read from LDS by the transposing ds_read_b64_tr_b4: seven
// products per block of 16 columns.  One wave walks down a strip of columns
// (256 four-bit, 128 Blume-Capel or 512 one-bit cells of a plane row) in tiles of 32 rows, its
// fragments of the tile before in registers, so every cell is read from
// memory once and staged in LDS once.  The waves of a workgroup take strips
// side by side and read their neighbours' edge cells from LDS.
//
// What it replaced counted xors of bit words, 2 to 3 VALU instructions per
// 32 pairs of 64 distances, and was bound by VALU issue.  Measured, before and
// after, the B/M/Q work included: 4-bit Ising L = 2^17 4.00 -> 1.96 ms (8.6 GB of
// lattice, 10.3 read with the strips' edge lines: 5.2 TB/s, bound by memory reads:
// a kernel that only loads in this pattern takes 1.42), 1-bit L = 2^16 0.85 -> 0.30 ms (matrix and VALU issue),
// Blume-Capel L = 2^15 0.87 -> 0.17 ms (0.54 GB: 3.1 TB/s; VALU issue beside
// the reads).  Edge cells read from memory by each wave, not each workgroup,
// made it 2.9 ms at L = 2^17.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "measure_device.h"

namespace mcl {
namespace {

// Order of a wave's accesses to its own LDS words (they execute in order; the
// compiler must not move a lane's read above another lane's write).
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

constexpr int kTileRows = 32;               // rows of a tile: two blocks of 16
// Tiles of a unit (a wave's run down its strip).  An accumulator takes at most
// 16 products of at most 128 per tile: below 2^22 for 2048 tiles.  Runs of 64,
// several rounds of workgroups at L = 2^17, end more evenly than one round of
// 512 tiles each: one measurement 2.36 against 2.57 ms (runs of 32 2.33, but
// Blume-Capel L = 2^15 and 1-bit L = 2^16, one round with runs of 64, 2% slower).
constexpr int kMaxTiles = 64;

// 1-bit strips of 512 cells need 16 to 24 registers more than the 256 that two
// waves per SIMD leave and keep them in scratch (68 to 100 bytes a lane): a
// quench of L = 2^16 with three measurements takes 6.39 ms, without a spill, one
// wave per SIMD, 6.54.
// Strips: 256 four-bit cells (with 128, half a row of fragments per lane, the
// measurement at L = 2^17 takes 2.50 against 2.36 ms), but 128 for
// Blume-Capel, whose two bit planes of 256 need 148 registers more than there
// are (0.41 against 0.17 ms at L = 2^15).
template <int MODEL>
struct Shape {
    static constexpr int CB = MODEL == 2 ? 1 : 4;
    static constexpr int NB = MODEL == 1 ? 2 : 1;           // bit planes of a cell
    static constexpr int NC = MODEL == 2 ? 4 : MODEL == 1 ? 1 : 2;  // 32-cell vectors per lane, row block and U_p
    static constexpr int NV = 4 * NC;                       // vectors of a strip row
    static constexpr int RAW = MODEL == 2 ? 1 : NC;         // 16-byte loads for them
    static constexpr int WAVES = MODEL == 2 ? 2 : 4;        // a workgroup's strips, side by side
    static constexpr int ROWB = WAVES * NV * 16 + 16;       // LDS bytes of its row (16 for halo cells)
    static constexpr int CELLB = 2 * kTileRows * ROWB + 16;
    static constexpr bool HALF = NV == 4;                   // a strip row gives half a T word
    static constexpr int TW = HALF ? 1 : NV / 8;            // (half) T words of a strip row
    static constexpr int TB = NB * TW * 16 * 16 * 4;        // T words of 16 row blocks
    static constexpr int RB = MODEL == 0 ? 16 * 16 * 4 : 0; // packed words of 16 sampled rows
    // vector of lane group h at index c
    static __device__ __forceinline__ int vec(int h, int c) { return MODEL == 2 ? 4 * h + c : 4 * c + h; }
    // cell (0 .. 15) at nibble j of a staged block of 16 (the order of expand())
    static __device__ __forceinline__ int cell(int j) { return MODEL == 2 ? 4 * (j & 3) + (j >> 2) : j; }
};

// Bit `BIT` of each nibble of a cleaned vector, cell 8 d + k at bit 4 k + d.
template <int MODEL, int BIT>
__device__ __forceinline__ uint32_t gather(const uint4& v)
{
    if (MODEL == 0) return (v.x >> 1) | shl_or<1>(shl_or<1>(v.w, v.z), v.y);     // (bits masked already)
    const uint32_t s0 = BIT ? v.x >> 1 : v.x, s1 = BIT ? v.y : v.y << 1;
    const uint32_t s2 = v.z << (2 - BIT), s3 = v.w << (3 - BIT);
    return bit_select(0x11111111u, s0, bit_select(0x22222222u, s1, bit_select(0x88888888u, s3, s2)));
}

// Bits of the cells i + 1 (i - 1) of bits z, `next` (`prev`) the fp4 word of
// the 8 cells after (before) them, whose bit BIT of the first (last) nibble
// comes in.  4-bit cells in gather() order, 1-bit cells in their own.
template <int MODEL, int BIT>
__device__ __forceinline__ uint32_t cell_right(uint32_t z, uint32_t next)
{
    if (MODEL == 2) return funnel(next >> 1, z, 1);
    return funnel(bit_select(0x7u, z >> 1, next << (3 - BIT)), z, 4);
}

template <int MODEL, int BIT>
__device__ __forceinline__ uint32_t cell_left(uint32_t z, uint32_t prev)
{
    if (MODEL == 2) return funnel(z, prev << 2, 31);
    return funnel(z, bit_select(0x10000000u, BIT ? prev >> 1 : prev, z << 1), 28);
}

// Row y - 1's value of x: lane m takes lane m - 1 of its 16, lane 0 lane 15
// of the block above; and row y + 1's, lane 15 from lane 0 of the block below.
__device__ __forceinline__ uint32_t row_above(uint32_t x, uint32_t above)
{
    const int old = __builtin_amdgcn_update_dpp(0, (int)above, 0x121, 0xF, 0xF, true);      // row_ror:1
    return (uint32_t)__builtin_amdgcn_update_dpp(old, (int)x, 0x111, 0xF, 0xF, false);      // row_shr:1
}

__device__ __forceinline__ uint32_t row_below(uint32_t x, uint32_t below)
{
    const int old = __builtin_amdgcn_update_dpp(0, (int)below, 0x12F, 0xF, 0xF, true);      // row_ror:15
    return (uint32_t)__builtin_amdgcn_update_dpp(old, (int)x, 0x101, 0xF, 0xF, false);      // row_shl:1
}

// x or-ed with the value GROUP lanes away (lane ^ GROUP; GROUP 16 or 32).
template <int GROUP>
__device__ __forceinline__ uint32_t or_groups(uint32_t x)
{
    const auto s = GROUP == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                               : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return s[0] | s[1];
}

// Bits of one row block of the wave, and of the block before what the sites
// of that block still need once the row below their last one is known.
template <int MODEL>
struct Bits {
    uint32_t z[2][Shape<MODEL>::NB];      // U_0, U_1: [s = +1] (Blume-Capel: [n = 2], [n = 1])
    uint32_t side[2][Shape<MODEL>::NB];   // the horizontal neighbour in the other vector position: p = 0 left, p = 1 right
    uint32_t up[2][Shape<MODEL>::NB];     // the row above
};

// The four neighbours of the sites o of one U_p: adds to the histogram bins.
// Ising: m of four neighbours differ; the set bits of m, and where m = 3.
template <int MODEL>
__device__ __forceinline__ void bins(const uint32_t* o, const uint32_t* a, const uint32_t* b, const uint32_t* c,
                                     const uint32_t* d, uint32_t (&hist)[9])
{
    if (MODEL != 1) {
        const uint32_t d0 = a[0] ^ o[0], d1 = b[0] ^ o[0], d2 = c[0] ^ o[0], d3 = d[0] ^ o[0];
        const uint32_t u1 = d0 & d1, t1 = d0 ^ d1, u2 = d2 & d3, t2 = d2 ^ d3;
        const uint32_t m0 = t1 ^ t2, m1 = (u1 ^ u2) | (t1 & t2);
        hist[0] = bcnt_acc(m0, hist[0]);
        hist[1] = bcnt_acc(m1, hist[1]);
        hist[2] = bcnt_acc(u1 & u2, hist[2]);
        hist[3] = bcnt_acc(m0 & m1, hist[3]);
        return;
    }
    // t = sigma h + 4 = the sum of the neighbours' n, n -> 2 - n where
    // sigma = -1: hi and lo bits of four numbers through full adders
    constexpr int LO = MODEL == 1 ? 1 : 0;
    const uint32_t neg = ~(o[0] | o[LO]), nz = ~o[LO];
    const uint32_t* n[4] = {a, b, c, d};
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        l[i] = n[i][LO];
        h[i] = bit_select(neg, ~(n[i][0] | n[i][LO]), n[i][0]);
    }
    const auto maj = [](uint32_t x, uint32_t y, uint32_t z) { return (x & y) | (z & (x | y)); };
    const uint32_t s1 = xor3(l[0], l[1], l[2]), c1 = maj(l[0], l[1], l[2]);
    const uint32_t b0 = s1 ^ l[3], c2 = s1 & l[3];
    const uint32_t t1 = xor3(h[0], h[1], h[2]), e1 = maj(h[0], h[1], h[2]);
    const uint32_t t2 = xor3(h[3], c1, c2), e2 = maj(h[3], c1, c2);
    const uint32_t b1 = t1 ^ t2, e3 = t1 & t2;
    const uint32_t b2 = xor3(e1, e2, e3), b3 = maj(e1, e2, e3);
    const uint32_t q[4] = {nz & ~b0 & ~b1, nz & b0 & ~b1, nz & ~b0 & b1, nz & b0 & b1};
#pragma unroll
    for (int k = 0; k < 8; ++k) hist[k] = bcnt_acc(k < 4 ? q[k] & ~(b2 | b3) : q[k - 4] & b2, hist[k]);
    hist[8] = bcnt_acc(nz & b3, hist[8]);
}

// A unit is a strip for each wave and a run of tiles down them; unit u is
// u % nstrips, run u / nstrips, and the runs split the tiles evenly.  The
// sites of a unit's histogram are the rows from 16 above its first to 16
// above its last (the row below a site has to be known), so a tile above the
// run is read first, for its rows' bits and fragments only.
// Cx, Cy: 33 sums each.  acc (or null): #(+1) to [2], #(0) to [4], the bins of
// sigma h to [5 .. 13], units with a cell that holds no spin to [14].
// tb (or null): T bits; rb (or null; 4-bit Ising): residue rows (internal.h).
// RAGGED: the last strip has fewer columns than the others.  TBITS: tb is
// given (and rb for 4-bit Ising).
template <int MODEL, bool RAGGED, bool TBITS>
__global__ __launch_bounds__(64 * Shape<MODEL>::WAVES) __attribute__((amdgpu_waves_per_eu(2))) void pass_kernel(
    const uint32_t* __restrict__ planes, uint32_t L, uint32_t nstrips, uint32_t nruns, int64_t* __restrict__ Cx,
    int64_t* __restrict__ Cy, int64_t* __restrict__ acc, uint32_t* __restrict__ tb, uint32_t* __restrict__ rb)
{
    using S = Shape<MODEL>;
    constexpr int NB = S::NB, NC = S::NC, RAW = S::RAW;
    __shared__ __align__(16) char smem[S::CELLB];
    __shared__ uint32_t bits[S::WAVES][(S::TB + S::RB) / 4 + 1];
    __shared__ unsigned long long sums[66 + 12];
    for (int i = threadIdx.x; i < 78; i += blockDim.x) sums[i] = 0;
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, h = lane >> 4;
    char* cells = smem + 16;                                    // slot (p, r) at (32 p + r) ROWB
    char* strip_cells = cells + wave * (S::NV * 16);            // the wave's columns of slot (0, 0)
    uint32_t* tbuf = bits[wave];
    uint32_t* zbuf = tbuf + S::TB / 4;
    const uint32_t rowB = (L >> 4) * S::CB;                     // bytes of a plane row
    const uint32_t Q = rowB >> 4;                               // its 16-byte units
    const size_t planeB = (size_t)L * rowB;
    const char* base = reinterpret_cast<const char*>(planes);
    constexpr uint32_t SQ = S::RAW * 4;                         // units of a strip row
    const uint32_t NS = L >> 4;

    // workgroup ids go round-robin to the 8 XCDs: XCD x takes the x-th eighth
    // of the units in order, so neighbouring strips, which read each other's
    // edge lines, meet in one L2
    const uint32_t nb = gridDim.x;
    const uint32_t blk0 = (nb & 7u) == 0 ? (blockIdx.x & 7u) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    for (uint32_t unit = blk0; unit < nstrips * nruns; unit += nb) {
        const uint32_t run = unit / nstrips, strip = (unit - run * nstrips) * S::WAVES + wave;
        const uint32_t RT = L / kTileRows;
        const uint32_t t0 = (uint32_t)((uint64_t)run * RT / nruns), t1 = (uint32_t)((uint64_t)(run + 1) * RT / nruns);
        const uint32_t q0 = strip * SQ;
        const uint32_t nq = RAGGED ? (q0 < Q ? min(SQ, Q - q0) : 0u) : SQ;      // units that the row has
        const int nv = MODEL == 2 ? 4 * (int)nq : (int)nq;      // 32-cell vectors
        // the workgroup's columns, for its halo cells
        const uint32_t w0 = (strip - wave) * SQ, wq = min(S::WAVES * SQ, Q - w0);
        // lane's addresses: its units of row m of the two U_p, and for wave 0
        // the cells left of the workgroup's columns in row `lane & 31` of
        // U_(lane >> 5), for wave 1 those right of them
        const char* src[2][RAW];
        bool has[RAW];
#pragma unroll
        for (int c = 0; c < RAW; ++c) {
            const uint32_t u = MODEL == 2 ? (uint32_t)h : (uint32_t)(4 * c + h);
            has[c] = !RAGGED || u < nq;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                src[p][c] = base + ((p + m) & 1) * planeB + (size_t)m * rowB + (size_t)(has[c] ? q0 + u : 0u) * 16;
        }
        bool valid[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) valid[c] = !RAGGED || S::vec(h, c) < nv;
        const int hr = lane & 31, hp = lane >> 5;
        const uint32_t hq = wave == 0 ? (w0 == 0 ? Q : w0) - 1 : (w0 + wq == Q ? 0u : w0 + wq);
        const char* hrow = base + ((hp + hr) & 1) * planeB + (size_t)hr * rowB + (size_t)hq * 16 + (wave == 0 ? 8 : 0);

        v4f y[3], Ed, En, Od, O01, O10;
        y[0] = y[1] = y[2] = Ed = En = Od = O01 = O10 = v4f{0.f, 0.f, 0.f, 0.f};
        uint32_t hist[9], n2 = 0, n1 = 0, bad = 0, both = 0;
#pragma unroll
        for (int k = 0; k < 9; ++k) hist[k] = 0;
        uint4 next[2][2][RAW];                                  // row block, p, unit
        uint2 halo;
        const auto load = [&](uint32_t tile) {
            const size_t off = (size_t)tile * kTileRows * rowB;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int c = 0; c < RAW; ++c)
                        next[b][p][c] = *reinterpret_cast<const uint4*>(src[p][c] + off + (size_t)(16 * b) * rowB);
            if (wave < 2) halo = *reinterpret_cast<const uint2*>(hrow + off);
        };
        uint4 even[2][2][RAW], odd[2][2][RAW];                  // fragments of the last two tiles
        Bits<MODEL> pb[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int k = 0; k < NB; ++k) pb[c].z[p][k] = pb[c].side[p][k] = pb[c].up[p][k] = 0;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int c = 0; c < RAW; ++c) even[b][p][c] = odd[b][p][c] = make_uint4(0, 0, 0, 0);
        const auto frag = [](const uint4 (&v)[RAW], int c) {
            return MODEL == 2 ? expand(pick(v[0], c)) : v[MODEL == 2 ? 0 : c];
        };
        uint32_t tfrom = 2 * t0;                                // first row block in tbuf and zbuf

        // one tile, its loads in `next` (then tile `after` is loaded), its cells
        // into cur, those of the tile above in prev; COUNT false for the tile
        // above the run, kept for its bits and fragments only
        const auto step = [&](auto counted, uint32_t at, uint32_t after, uint4 (&cur)[2][2][RAW],
                              const uint4 (&prev)[2][2][RAW]) {
            constexpr bool COUNT = decltype(counted)::value;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int c = 0; c < RAW; ++c) {
                        uint4 v = next[b][p][c];
                        if (RAGGED && !has[c]) v = make_uint4(0, 0, 0, 0);
                        if (MODEL != 2) {
                            v.x = clean<MODEL>(v.x, bad, both);
                            v.y = clean<MODEL>(v.y, bad, both);
                            v.z = clean<MODEL>(v.z, bad, both);
                            v.w = clean<MODEL>(v.w, bad, both);
                        }
                        cur[b][p][c] = v;
                    }
            uint2 edge = halo;
            uint32_t unused = 0;
            if (MODEL == 2) {
                const uint4 e = expand(edge.x);
                edge = make_uint2(e.x, wave == 0 ? (edge.y >> 31) << 29 : e.y);   // (left: the last cell at nibble 7)
            } else {
                edge.x = clean<MODEL>(edge.x, unused, unused);
                edge.y = clean<MODEL>(edge.y, unused, unused);
            }
            __syncthreads();                                    // the tile before is done with
            // the next tile's loads, in flight over this one's work
            load(min(after, t1 - 1));
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        *reinterpret_cast<uint4*>(strip_cells + (32 * p + 16 * b + m) * S::ROWB + 16 * S::vec(h, c)) =
                            frag(cur[b][p], c);
            // (row r - 1's last word holds row r's left cell)
            if (wave == 0) *reinterpret_cast<uint32_t*>(cells + lane * S::ROWB - 4) = edge.y;
            if (RAGGED) __syncthreads();                        // (the right cells follow the last vector the row has)
            if (wave == 1)
                *reinterpret_cast<uint2*>(cells + lane * S::ROWB + 16 * (int)(MODEL == 2 ? 4 * wq : wq)) = edge;
            if constexpr (COUNT) {
                // along y: this tile's two blocks as targets
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const uint4 f0 = frag(cur[0][p], c), f1 = frag(cur[1][p], c);
                        const uint4 g0 = frag(prev[0][p], c), g1 = frag(prev[1][p], c);
                        y[0] = mfma_f4(f0, f0, y[0]);
                        y[1] = mfma_f4(g1, f0, y[1]);
                        y[2] = mfma_f4(g0, f0, y[2]);
                        y[0] = mfma_f4(f1, f1, y[0]);
                        y[1] = mfma_f4(f0, f1, y[1]);
                        y[2] = mfma_f4(g1, f1, y[2]);
                    }
            }
            __syncthreads();
            uint32_t nx[2][NC], pv[2][NC];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const char* row0 = strip_cells + (16 * b + m) * S::ROWB + 16 * S::vec(h, c);
                    nx[b][c] = *reinterpret_cast<const uint32_t*>(row0 + 16);
                    pv[b][c] = *reinterpret_cast<const uint32_t*>(row0 + 32 * S::ROWB - 4);
                }
            // B/M/Q, the histogram, T bits and residue rows
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                uint32_t tw[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) tw[k] = 0;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    Bits<MODEL> w;
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        if (MODEL == 2) {
                            w.z[p][0] = pick(cur[b][p][0], c);
                        } else {
                            w.z[p][0] = gather<MODEL, 1>(cur[b][p][MODEL == 2 ? 0 : c]);
                            if (NB == 2) w.z[p][NB - 1] = gather<MODEL, 0>(cur[b][p][MODEL == 2 ? 0 : c]);
                        }
                    }
                    w.side[0][0] = cell_left<MODEL, 1>(w.z[1][0], pv[b][c]);
                    w.side[1][0] = cell_right<MODEL, 1>(w.z[0][0], nx[b][c]);
                    if (NB == 2) {
                        w.side[0][NB - 1] = cell_left<MODEL, 0>(w.z[1][NB - 1], pv[b][c]);
                        w.side[1][NB - 1] = cell_right<MODEL, 0>(w.z[0][NB - 1], nx[b][c]);
                    }
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int k = 0; k < NB; ++k) w.up[p][k] = row_above(w.z[p][k], pb[c].z[p][k]);
                    if (COUNT && valid[c]) {
#pragma unroll
                        for (int p = 0; p < 2; ++p) {
                            uint32_t down[NB];
#pragma unroll
                            for (int k = 0; k < NB; ++k) down[k] = row_below(pb[c].z[p][k], w.z[p][k]);
                            bins<MODEL>(pb[c].z[p], pb[c].up[p], down, pb[c].z[1 - p], pb[c].side[p], hist);
                            n2 = bcnt_acc(w.z[p][0], n2);
                            if (NB == 2) n1 = bcnt_acc(w.z[p][NB - 1], n1);
                        }
                    }
                    if (TBITS) {
                        // sampled columns x = 0 mod 16: cells 0, 8, 16, 24 of U_0
                        uint32_t s[2] = {w.z[0][0], ~w.z[0][NB - 1]};
#pragma unroll
                        for (int k = 0; k < NB; ++k) {
                            uint32_t f = s[k] & 0xFu;
                            if (MODEL == 2) {
                                const uint32_t x = s[k] & 0x01010101u;
                                f = (x | (x >> 7) | (x >> 14) | (x >> 21)) & 0xFu;
                            }
                            tw[k] |= f << (4 * (S::vec(h, c) & 7));
                        }
                    }
                    if (TBITS && MODEL == 0 && m == 0) {
                        uint32_t* zw = zbuf + ((2 * at + b) & 15) * 16 + S::vec(h, c);
                        zw[0] = w.z[0][0];
                        zw[8] = w.z[1][0];
                    }
                    pb[c] = w;
                }
                if (TBITS) {
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        // the lane groups h that share the word
                        tw[k] = or_groups<16>(tw[k]);
                        if (S::TW == 1) tw[k] = or_groups<32>(tw[k]);
                        const int word = S::TW == 1 ? 0 : h >> 1;
                        if ((h & (S::TW == 1 ? 3 : 1)) == 0)
                            tbuf[(k * S::TW + word) * 256 + m * 16 + (int)((2 * at + b) & 15)] = tw[k];
                    }
                }
            }
            if constexpr (COUNT) {
                // along x: lane group h takes the blocks BPH h .. BPH h + BPH - 1
                // of the strip, its 32 rows of each: 128 rows in all
                constexpr int BPH = S::NV / 2;
                const auto column = [&](int p, int blk) {
                    return columns16(strip_cells + (32 * p + m) * S::ROWB + 8 * (BPH * h + blk), 16 * S::ROWB);
                };
                uint4 F0 = column(0, 0), F1 = column(1, 0);
#pragma unroll
                for (int blk = 0; blk < BPH; ++blk) {
                    const uint4 G0 = column(0, blk + 1), G1 = column(1, blk + 1);
                    uint4 A0 = F0, A1 = F1;
                    if (RAGGED && BPH * h + blk >= 2 * nv) A0 = A1 = make_uint4(0, 0, 0, 0);
                    Ed = mfma_f4(A0, F0, Ed);
                    En = mfma_f4(A0, G0, En);
                    Od = mfma_f4(A0, F1, Od);
                    O01 = mfma_f4(A0, G1, O01);
                    O10 = mfma_f4(A1, G0, O10);
                    Ed = mfma_f4(A1, F1, Ed);
                    En = mfma_f4(A1, G1, En);
                    F0 = G0;
                    F1 = G1;
                }
            }
            if (COUNT && TBITS && (((2 * at + 1) & 15) == 15 || after == t1)) {
                // T words and residue words of row blocks [tfrom, 2 at + 2)
                const uint32_t from = tfrom & 15, to = (2 * at + 1) & 15, b0 = (2 * at) & ~15u;
                wave_order();
                const uint32_t NSW = L >> 9;
#pragma unroll 1
                for (int k = 0; k < NB * S::TW; ++k) {
                    const uint32_t word = S::HALF ? strip >> 1 : strip * S::TW + (k % S::TW);
                    if (word >= NSW) continue;
                    uint32_t* out = tb + (size_t)(k / S::TW) * L * NSW + (size_t)word * L;
#pragma unroll 1
                    for (uint32_t i = lane; i < 256; i += 64) {
                        const uint32_t rho = i >> 4, s = i & 15;
                        if (s < from || s > to) continue;
                        if (S::HALF)
                            reinterpret_cast<uint16_t*>(out + rho * NS + b0 + s)[strip & 1u] = (uint16_t)tbuf[k * 256 + i];
                        else
                            out[rho * NS + b0 + s] = tbuf[k * 256 + i];
                    }
                }
                if (MODEL == 0 && strip < NSW) {
#pragma unroll 1
                    for (uint32_t i = lane; i < 256; i += 64) {
                        const uint32_t s = i >> 4, rho = i & 15;
                        const uint32_t* zw = zbuf + s * 16 + 8 * (rho & 1);
                        uint32_t w = 0;
#pragma unroll
                        for (int v = 0; v < 8; ++v) w |= ((zw[v] >> (4 * (rho >> 1))) & 0xFu) << (4 * v);
                        if (s >= from && s <= to) rb[((size_t)(b0 + s) * NSW + strip) * 16 + rho] = w;
                    }
                }
                wave_order();
                tfrom = 2 * at + 2;
            }
        };
        load(t0 == 0 ? RT - 1 : t0 - 1);
        step(std::false_type(), t0 == 0 ? RT - 1 : t0 - 1, t0, odd, even);
        for (uint32_t tile = t0;;) {
            step(std::true_type(), tile, tile + 1, even, odd);
            if (++tile == t1) break;
            step(std::true_type(), tile, tile + 1, odd, even);
            if (++tile == t1) break;
        }

        // the unit's sums: entry (i, j) of a product by the distance of its cells
        const auto add = [&](int idx, float v) {
            if (v != 0.f) atomicAdd(&sums[idx], (unsigned long long)(long long)(4.f * v));
        };
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ra = 4 * h + i, dy = m - ra;              // rows
            if (dy >= 0) add(33 + dy, y[0][i]);
            add(33 + 16 + dy, y[1][i]);
            if (dy <= 0) add(33 + 32 + dy, y[2][i]);
            const int dx = S::cell(m) - S::cell(ra);            // columns of one U_p
            if (dx >= 0) add(2 * dx, Ed[i]);
            if (dx <= 0) add(32 + 2 * dx, En[i]);
            add(dx >= 0 ? 2 * dx + 1 : -2 * dx - 1, Od[i]);
            if (dx < 0) add(33 + 2 * dx, O01[i]);
            if (dx <= 0) add(31 + 2 * dx, O10[i]);
        }
        int pairs = 0;                                          // vectors of U_0 and U_1 that the lane holds
#pragma unroll
        for (int c = 0; c < NC; ++c) pairs += valid[c] ? 1 : 0;
        // the wave's sums (below 2^31: kMaxTiles tiles of 2^15 cells at most)
        const int sites = wave_sum_i32(pairs * 128 * (int)(t1 - t0));
        const int s2 = wave_sum_i32((int)n2), s1 = MODEL == 1 ? wave_sum_i32((int)n1) : 0;
        int t[9];
        if (MODEL == 1) {
#pragma unroll
            for (int k = 0; k < 9; ++k) t[k] = wave_sum_i32((int)hist[k]);
            t[4] += s1;                                         // sigma = 0: t = 4
        } else {
            int e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = wave_sum_i32((int)hist[k]);
            t[6] = e[0] - e[3];                                 // 1, 2, 3, 4 neighbours differ
            t[4] = e[1] - e[3];
            t[2] = e[3];
            t[0] = e[2];
            t[8] = sites - t[6] - t[4] - t[2] - t[0];
            t[1] = t[3] = t[5] = t[7] = 0;
        }
        const int worst = __any((bad | (both & 0x22222222u)) != 0);
        // every distance gets -2 sum n + N
        const int64_t rest = (int64_t)sites - 2 * (2 * (int64_t)s2 + s1);
        for (int i = lane; i < 66; i += 64) atomicAdd(&sums[i], (unsigned long long)rest);
        int64_t v = 0;
        if (lane == 0) v = s2;
        if (lane == 1) v = s1;
#pragma unroll
        for (int k = 0; k < 9; ++k)
            if (lane == 2 + k) v = t[k];
        if (lane == 11) v = worst;
        if (v != 0) atomicAdd(&sums[66 + lane], (unsigned long long)v);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 78; i += blockDim.x) {
        const unsigned long long s = sums[i];
        if (s == 0) continue;
        if (i < 66) atomicAdd((unsigned long long*)(i < 33 ? &Cx[i] : &Cy[i - 33]), s);
        else if (acc) atomicAdd((unsigned long long*)&acc[i == 66 ? 2 : i == 67 ? 4 : i - 63], s);
    }
}

}  // namespace

hipError_t launch_pass(const Geom& g, int model, int64_t* Cx, int64_t* Cy, int64_t* acc, uint32_t* tbits,
                       uint32_t* rbits, hipStream_t s)
{
    if ((rbits != nullptr) != (tbits != nullptr && model == 0)) return hipErrorInvalidValue;
    if (tbits && (g.L < 512 || (g.L & (g.L - 1)) != 0)) return hipErrorInvalidValue;
    const int64_t per = model == 0 ? 8 : 4;                       // 16-byte units of a strip row
    const uint32_t waves = model == 2 ? 2 : 4;
    const uint32_t nstrips = (uint32_t)((g.Q + per * waves - 1) / (per * waves));
    const int64_t RT = g.L / kTileRows;
    // two waves per SIMD of 256 CUs while there are tiles for them, and runs of
    // no more than kMaxTiles.  (A run reads one tile above it: runs of two
    // tiles read half as much more, of one twice, but a small lattice is in
    // cache and waits for its longest run.)
    const uint32_t cap = measure_grid_cap(2048 / waves);
    int64_t runs = std::max<int64_t>(1, std::min<int64_t>(cap / nstrips, RT));
    runs = std::max<int64_t>(runs, (RT + kMaxTiles - 1) / kMaxTiles);
    const dim3 grid(measure_grid_cap(nstrips * (uint32_t)runs));
    const auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * waves), 0, s, g.plane0, (uint32_t)g.L, nstrips, (uint32_t)runs, Cx, Cy,
                           acc, tbits, rbits);
    };
    const bool ragged = g.Q % (per * waves) != 0;
    const auto pick = [&](auto rt, auto r, auto t) {
        if (tbits) ragged ? go(rt) : go(t);
        else go(r);
    };
    if (model == 0) pick(pass_kernel<0, true, true>, pass_kernel<0, true, false>, pass_kernel<0, false, true>);
    else if (model == 1) pick(pass_kernel<1, true, true>, pass_kernel<1, true, false>, pass_kernel<1, false, true>);
    else pick(pass_kernel<2, true, true>, pass_kernel<2, true, false>, pass_kernel<2, false, true>);
    return hipGetLastError();
}

}  // namespace mcl
