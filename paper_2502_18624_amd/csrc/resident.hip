// Small lattices, many sweeps, one launch (gfx950): a workgroup holds both
// colour planes of its lattice in LDS and runs every sweep of the call on
// them, reading and writing the lattice in memory once.
//
// A half-sweep of a small lattice as a launch of its own is bound by latency:
// the launch, the loads of a thread's rows and their chain of row steps (L =
// 256: 4.4 us for 2^15 updates, which are 0.012 us of the chip's VALU work).
// Here a half-sweep costs a barrier and its work on one compute unit, bound by
// VALU issue; the draws are keyed by (seed, sweep, site), so the lattice is
// the same.  512 replicas of L = 256, 16 sweeps: 280 us, 79% of the VALU rate
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

// Dynamic LDS of a launch, beside the kernels' tables.
constexpr size_t kMostLds = 150 * 1024;

// The largest lattices that trapezoid launches are for, us per sweep at 32
// sweeps, against one launch per half-sweep: L = 7168 27.6 against about 29,
// L = 8192 33.6 against 33.9 and 34.7 against 34.0 at three sweeps; 1-bit
// L = 12288 42.6 against 50.4 (L = 16384 does not fit LDS in 256 tiles).
constexpr int64_t kTrapezoidMaxL = 7168, kTrapezoidMaxLutL = 12288;
// The largest whose single sweeps take a word per thread: L = 3072 12.1 against
// 13.1 us (Blume-Capel 15.4, 16.9), 4096 19.2 against 13.6; 1-bit 4096 11.5
// against 27.6.
constexpr int64_t kHalfWordsMaxL = 3072, kHalfWordsMaxLutL = 4096;

// Parameters of the updates of one lattice (tables in LDS).
struct Rule {
    uint32_t k0, k1, T4, T8;        // (T8: the 1-bit table's eighth threshold)
    const uint2* bc;                // Blume-Capel
    const uint2* buckets;           // 1-bit cells
    const uint32_t* lut;
    uint32_t kmax;
};

// Update of the vector q (of Q) of row y, colour c, sweep t, in LDS: its row at
// `own`, the other colour's rows y - 1, y, y + 1 at up, row, dn.  (Both sides'
// neighbour words and a select per word: one copy of the update's code, and a
// wave may hold rows of both parities.)
template <int MODEL>
__device__ __forceinline__ void update_vector(const Rule& u, char* own, const char* up, const char* row, const char* dn,
                                              uint32_t q, uint32_t Q, uint32_t y, uint32_t L, uint32_t c, uint32_t t)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    uint4* at = reinterpret_cast<uint4*>(own) + q;
    const uint4 src = *at, a = dev::load_row(up, 16 * q), b = dev::load_row(dn, 16 * q), mid = dev::load_row(row, 16 * q);
    const bool odd = ((y + c) & 1u) != 0;
    const uint32_t side = odd ? (q + 1 == Q ? 0u : 16 * q + 16) : (q == 0 ? 16 * Q : 16 * q) - 4;
    const uint32_t halo = *reinterpret_cast<const uint32_t*>(row + side);
    const uint32_t kv = y * (L >> 1) + (128 / CB) * q;                  // in-colour index of cell 0
    if (MODEL == 0) {
        *at = dev::ising_vec<0>(src, a, b, mid, halo, odd, kv >> 2, 0u, t, c, u.k0, u.k1, 0u, u.T4, u.T8);
    } else if (MODEL == 2) {
        *at = dev::lut_vec<0>(src, a, b, mid, halo, odd, kv, t, c, u.k0, u.k1, 0u, u.buckets, u.lut, u.T8, u.kmax);
    } else {
        const Philox4 p = philox4x32_10(kv >> 7, 0u, t, 2u + c, u.k0, u.k1);
        *at = dev::bc_vec<0>(src, a, b, mid, halo, odd, kv >> 2, 0u, philox_word(p, (int)((kv >> 5) & 3)), t, c, u.k0,
                             u.k1, 0u, u.bc);
    }
}

// ---------------------------------------------------------------------------
// The same word by word, for the steps that have too few vectors for a
// compute unit's waves: 8 four-bit cells (two accept blocks) or 32 one-bit
// cells per thread.  An acceptance bit goes straight to its cell's nibble, a
// select and half an or instead of an add per draw and threshold, since the
// carry chain's order (sweep_device.h) belongs to four words at once: about
// 18 VALU a cell against 15 for Ising.
// ---------------------------------------------------------------------------
// Blume-Capel: a generator block of proposal bits serves 16 words, so the
// workgroup draws a half-sweep's blocks during the one before, into LDS:
// row r (row y of the lattice) has the row_blocks(Q) blocks from (y Q) / 4 on.
__host__ __device__ __forceinline__ uint32_t row_blocks(uint32_t Q) { return (Q + 6) >> 2; }

// v / Q of v < 2^32 / Q, as the high word of v times this (Q > 1).
__device__ __forceinline__ uint32_t reciprocal(uint32_t Q) { return 0xFFFFFFFFu / Q + 1; }
__device__ __forceinline__ uint32_t quotient(uint32_t v, uint32_t Q, uint32_t recip) { return Q == 1 ? v : __umulhi(v, recip); }

// Row first + r of a lattice of L rows (first < 2 L, r < L).
__device__ __forceinline__ uint32_t row_of(uint32_t first, uint32_t r, uint32_t L)
{
    uint32_t y = first + r;
    y = y >= L ? y - L : y;
    return y >= L ? y - L : y;
}

// The proposal blocks of rows [lo, hi) (from row `first` on), colour c, sweep t.
__device__ __forceinline__ void draw_proposals(uint32_t* bits, uint32_t lo, uint32_t hi, uint32_t first, uint32_t L,
                                               uint32_t Q, uint32_t c, uint32_t t, uint32_t k0, uint32_t k1)
{
    const uint32_t nb = row_blocks(Q), recip = reciprocal(nb), total = (hi - lo) * nb;
    // (from the last thread down: the first ones take a last, partly filled
    // round of the words)
    for (uint32_t i = blockDim.x - 1 - threadIdx.x; i < total; i += blockDim.x) {
        const uint32_t dr = quotient(i, nb, recip), r = lo + dr;
        const Philox4 p = philox4x32_10(((row_of(first, r, L) * Q) >> 2) + (i - dr * nb), 0u, t, 2u + c, k0, k1);
        reinterpret_cast<uint4*>(bits)[r * nb + (i - dr * nb)] = make_uint4(p.v0, p.v1, p.v2, p.v3);
    }
}

// The word of proposal bits that holds those of in-colour index kv, from the
// proposal blocks of row y.
__device__ __forceinline__ uint32_t proposal_word(const uint32_t* props, uint32_t kv, uint32_t y, uint32_t Q)
{
    return props[(kv >> 5) - ((y * Q) & ~3u)];
}

// `proposals(kv)`: the word of proposal bits that holds those of index kv
// (Blume-Capel).  EXACT: 1-bit cells by the exact table search only.
template <int MODEL, bool EXACT = false, class P>
__device__ __forceinline__ void update_word(const Rule& u, char* own, const char* up, const char* row, const char* dn,
                                            uint32_t w, uint32_t W, uint32_t y, uint32_t L, uint32_t c, uint32_t t,
                                            const P& proposals)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    const auto at = [&](const char* r, uint32_t i) { return reinterpret_cast<const uint32_t*>(r)[i]; };
    const bool odd = ((y + c) & 1u) != 0;
    const uint32_t s = at(own, w), a = at(up, w), b = at(dn, w), mid = at(row, w);
    const uint32_t side = at(row, odd ? (w + 1 == W ? 0u : w + 1) : (w == 0 ? W : w) - 1);
    const uint32_t hs = odd ? funnel(side, mid, CB) : funnel(mid, side, 32 - CB);
    const uint32_t kv = y * (L >> 1) + (32 / CB) * w;                   // in-colour index of cell 0
    uint32_t res;
    if (MODEL == 2) {
        const uint32_t d0 = a ^ s, d1 = b ^ s, d2 = mid ^ s, d3 = hs ^ s;
        const uint32_t t1 = d0 ^ d1, u1 = d0 & d1, t2 = d2 ^ d3, u2 = d2 & d3;
        const uint32_t eq4 = ~(d0 | d1 | d2 | d3), eq3 = (t1 ^ t2) & ~(u1 | u2);
        const auto draw = [&](uint32_t stream) {
            if (!EXACT)
                return dev::lut_word_fast<0>(kv >> 2, t, stream, u.k0, u.k1, 0u, u.buckets, u.lut, u.T8, u.kmax);
            const uint32_t blk = kv >> 4;
            return dev::lut_word(philox4x32_10(blk, 0u, t, stream, u.k0, u.k1),
                                 philox4x32_10(blk + 1, 0u, t, stream, u.k0, u.k1), u.lut, u.T8, u.kmax);
        };
        const uint32_t e4 = draw(8u + 2u * c), e8 = draw(9u + 2u * c) & e4;
        res = ~(s ^ ((eq4 & ~e8) | (eq3 & ~e4)));
    } else {
        const Philox4 B[2] = {philox4x32_10(kv >> 2, 0u, t, c, u.k0, u.k1),
                              philox4x32_10((kv >> 2) + 1, 0u, t, c, u.k0, u.k1)};
        if (MODEL == 0) {
            uint32_t m4 = 0, m8 = 0;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const uint32_t r = philox_word(B[j >> 2], j & 3), bit = 2u << (4 * j);
                m4 |= r < u.T4 ? bit : 0u;
                m8 |= r < u.T8 ? bit : 0u;
            }
            uint32_t S = xad(a, s, 0x44444444u);
            S = xad(b, s, S);
            S = xad(mid, s, S);
            S = xad(hs, s, S);
            res = s ^ (((S >> 2) | (S & m4) | m8) & 0x22222222u);
        } else {
            const uint32_t pb = dev::spread8(proposals(kv) >> (kv & 31u));
            const uint32_t sum = a + b + mid + hs;
            const uint32_t key = s + s + pb;                            // n * 2 + b, at most 5 per nibble
            const uint32_t ev = ((key & 0x0F0F0F0Fu) << 4) | (sum & 0x0F0F0F0Fu);      // cells 0, 2, 4, 6 as bytes
            const uint32_t od = (key & 0xF0F0F0F0u) | ((sum >> 4) & 0x0F0F0F0Fu);      // cells 1, 3, 5, 7
            const uint32_t v = s + 0x11111111u + pb;                    // n + 1 + b in 1..4
            const uint32_t ge3 = ((v + 0x55555555u) & 0x88888888u) >> 3;
            const uint32_t nxt = v - shl_or<1>(ge3, ge3);               // mod 3
            uint32_t nacc = 0;                                          // -(accept bits)
#pragma unroll
            for (int j = 7; j >= 0; --j) {
                const uint2 e = u.bc[(((j & 1) ? od : ev) >> (8 * (j >> 1))) & 0xFFu];
                nacc = shl_add<1>(nacc, add_hi(philox_word(B[j >> 2], j & 3), ((uint64_t)e.y << 32) | e.x));
            }
            const uint32_t acc = dev::spread8(0u - nacc);
            const uint32_t mask = shl_opaque<4>(acc) - acc;             // 0xF in accepted nibbles
            res = (s & ~mask) | (nxt & mask);
        }
    }
    reinterpret_cast<uint32_t*>(own)[w] = res;
}

// LDS: the two planes, then the model's table (`extra`: 1-bit cells the
// buckets, Blume-Capel word by word the proposals of two half-sweeps).
template <int MODEL, bool WORDS>
__device__ __forceinline__ void run_resident(char* lds, uint32_t* extra, uint32_t* planes, uint32_t L, uint32_t t,
                                             uint32_t n, const Rule& rule)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    const uint32_t rowB = (L >> 4) * CB, Q = rowB >> 4, planeB = L * rowB;
    uint4* cells = reinterpret_cast<uint4*>(lds);
    uint4* mem = reinterpret_cast<uint4*>(planes);
    for (uint32_t i = threadIdx.x; i < planeB / 8; i += blockDim.x) cells[i] = mem[i];
    __syncthreads();
    const uint32_t U = WORDS ? 4 * Q : Q, units = U * L, recip = reciprocal(U);
    const uint32_t nb = row_blocks(Q);
    if (WORDS && MODEL == 1) {
        draw_proposals(extra, 0, L, 0, L, Q, 0, t, rule.k0, rule.k1);
        __syncthreads();
    }
    for (uint32_t s = 0; s < n; ++s, ++t)
        for (uint32_t c = 0; c < 2; ++c) {
            char* own = lds + c * planeB;
            const char* oth = lds + (1 - c) * planeB;
            for (uint32_t v = threadIdx.x; v < units; v += blockDim.x) {
                const uint32_t y = quotient(v, U, recip), q = v - y * U;
                const char* up = oth + (y == 0 ? L - 1 : y - 1) * rowB;
                const char* dn = oth + (y + 1 == L ? 0 : y + 1) * rowB;
                if (WORDS)
                    update_word<MODEL>(rule, own + y * rowB, up, oth + y * rowB, dn, q, U, y, L, c, t,
                                       [&](uint32_t kv) { return proposal_word(extra + (c * L + y) * nb * 4, kv, y, Q); });
                else
                    update_vector<MODEL>(rule, own + y * rowB, up, oth + y * rowB, dn, q, Q, y, L, c, t);
            }
            if (WORDS && MODEL == 1)
                draw_proposals(extra + (1 - c) * L * nb * 4, 0, L, 0, L, Q, 1 - c, t + c, rule.k0, rule.k1);
            __syncthreads();
        }
    for (uint32_t i = threadIdx.x; i < planeB / 8; i += blockDim.x) mem[i] = cells[i];
}

// LDS tables of the models of a launch.
struct ResidentLds {
    dev::BCLds bc;
    uint32_t lut[16];
};

template <int MODEL, bool WORDS>
__device__ __forceinline__ void resident(ResidentLds& tabs, const GroupDesc& d, uint32_t t, uint32_t n,
                                         const LutTable& lt)
{
    extern __shared__ __align__(16) char lds[];
    const uint32_t L = d.L;
    uint2* B = reinterpret_cast<uint2*>(lds + (size_t)L * L / (MODEL == 2 ? 8 : 2));      // after the planes
    if (MODEL == 2) {
        if (threadIdx.x < 16) tabs.lut[threadIdx.x] = lt.T[threadIdx.x];
        for (uint32_t b = threadIdx.x; b < (uint32_t)dev::kLutBuckets; b += blockDim.x) {
            const uint64_t A = dev::lut_bucket_addend(lt.T, lt.kmax, b);
            B[b] = make_uint2((uint32_t)A, (uint32_t)(A >> 32));
        }
    }
    const Rule rule{d.k0, d.k1, d.T4, MODEL == 2 ? lt.T[8] : d.T8, tabs.bc.e, B, tabs.lut, lt.kmax};
    run_resident<MODEL, WORDS>(lds, reinterpret_cast<uint32_t*>(B), d.plane0, L, t, n, rule);
}

// One lattice, its tables passed by value; word by word, as its vectors are too
// few for 1024 threads (L = 64 1.2 us a sweep, by vectors 2.5).
template <int MODEL>
__global__ __launch_bounds__(kMaxThreads) void resident_kernel(GroupDesc d, uint32_t n, BCTable bc, LutTable lt)
{
    __shared__ ResidentLds tabs;
    if (MODEL == 1) dev::load_bc_table(tabs.bc, bc);
    resident<MODEL, true>(tabs, d, d.t0, n, lt);
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
        resident<0, false>(tabs, d, d.t0 + s0, end - s0, lt);
    } else if (d.model == 1u) {
        dev::load_bc_table(tabs.bc, bc_tables + (size_t)d.tab * 96u);
        resident<1, false>(tabs, d, d.t0 + s0, end - s0, lt);
    } else {
        const LutRec* rec = luts + d.tab;
#pragma unroll
        for (int k = 0; k < 16; ++k) lt.T[k] = __builtin_amdgcn_readfirstlane(rec->T[k]);
        lt.kmax = __builtin_amdgcn_readfirstlane(rec->kmax);
        resident<2, false>(tabs, d, d.t0 + s0, end - s0, lt);
    }
}

// ---------------------------------------------------------------------------
// Several sweeps of a lattice in two launches, in place, without redundant
// work.  The rows are cut into tiles [a_i, a_i+1).  In the first launch a
// workgroup takes a tile into LDS and runs half-sweeps 0 .. k - 1 on it, each
// on one row less at either end, as far as its own rows determine them:
// half-sweep s (colour s & 1) on rows [a_i + s, a_i+1 - s).  In the second, a
// workgroup takes the rows around a cut and runs what was left: half-sweep s
// on rows [a_i - s, a_i + s).
//   First launch: half-sweep 0 reads colour 1 of the rows a_i - 1 and a_i+1,
// which no workgroup changes in this launch (half-sweep 1 starts a row
// inside); every later one reads rows of the tile only.
//   Second: half-sweep s reads the other colour on rows [a_i - s - 1, a_i + s],
// whose last update was half-sweep s - 1: of the rows inside by this
// workgroup, of the outermost two by the first launch, whose half-sweep
// s + 1 stayed a row further off.  With tiles of at least 2 k rows the
// rows of neighbouring cuts do not meet.
// A half-sweep is then a barrier and its work, not a launch and the latency of
// its loads: us per sweep at 32 sweeps, against launches per half-sweep, L =
// 256 3.6 against 8.1 (Blume-Capel 4.8, 11.8), 1024 4.9 against 8.5 (6.3, 12.4),
// 3008 9.2 against 12.6 (11.3, 15.8), 5120 16.4 against 21.0 (20.7, 25.8); 1-bit
// L = 1024 6.6 against 23.3, 4096 8.5 against 23.9, 8192 20.2 against 25.1.  The
// VALU work is about half of it from L = 3008 on; the rest is steps with less
// than a round of work for the waves.
//   That is a lattice alone on the chip.  Launches per half-sweep of lattices on
// several streams fill each other's gaps better than these do: eight streams, L =
// 2048 24.6 against 53.6 us for eight sweeps of a lattice (these against those),
// 3008 48 against 56, but 3584 64 against 54, 4096 84 against 58, 7168 220
// against 189 (Blume-Capel 2048 48 / 51, 3008 81 / 60, 4096 116 / 79; 1-bit 6144
// 79 / 86, 8192 133 / 122, 12288 343 / 277).  Part of it: two workgroups of 16
// waves share a compute unit only where the kernel takes no more than 80 scalar
// registers (the wave's trap registers make it 96, of 800 a SIMD), which the
// Blume-Capel and the vector forms exceed.  12 waves, or a limit on the
// registers, give four streams 1.2 to 1.4 times as much at L = 2560 .. 5120, but
// cost a lattice alone 1 to 5%.  Nothing tells a call what other streams do, so
// the rule is the lone lattice's; MCL_SWEEP_GRAPH=0 has the launches per
// half-sweep, and group_sweep takes many lattices together.
// ---------------------------------------------------------------------------
template <int MODEL, bool WORDS, bool CUTS>
__global__ __launch_bounds__(kMaxThreads) void trapezoid_kernel(uint32_t* __restrict__ planes, uint32_t L, uint32_t tiles,
                                                                uint32_t k, uint32_t t, uint32_t k0, uint32_t k1, uint32_t T4, uint32_t T8,
                                                                BCTable bc, LutTable lt,
                                                                const uint2* __restrict__ buckets)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    extern __shared__ __align__(16) char lds[];
    __shared__ ResidentLds tabs;
    const uint32_t rowB = (L >> 4) * CB, Q = rowB >> 4, W = rowB >> 2, recip = reciprocal(Q), recip_w = reciprocal(W);
    const uint32_t i = blockIdx.x;
    const uint32_t a = (uint32_t)((uint64_t)i * L / tiles), b = (uint32_t)((uint64_t)(i + 1) * L / tiles);
    // rows first .. first + rows - 1 (periodic) of both colours in LDS, one
    // colour after the other
    const uint32_t first = CUTS ? a + L - k : a + L - 1, rows = CUTS ? 2 * k : b - a + 2;
    const size_t planeB = (size_t)L * rowB;
    char* mem = reinterpret_cast<char*>(planes);
    const auto in_mem = [&](uint32_t c, uint32_t r, uint32_t q) {
        return reinterpret_cast<uint4*>(mem + c * planeB + (size_t)row_of(first, r, L) * rowB) + q;
    };
    const auto in_lds = [&](uint32_t c, uint32_t r, uint32_t q) {
        return reinterpret_cast<uint4*>(lds + (c * rows + r) * rowB) + q;
    };
    if (MODEL == 1) dev::load_bc_table(tabs.bc, bc);
    uint2* B = reinterpret_cast<uint2*>(lds + 2 * rows * rowB);
    if (MODEL == 2) {
        if (threadIdx.x < 16) tabs.lut[threadIdx.x] = lt.T[threadIdx.x];
        for (uint32_t v = threadIdx.x; v < (uint32_t)dev::kLutBuckets / 2; v += blockDim.x)
            reinterpret_cast<uint4*>(B)[v] = reinterpret_cast<const uint4*>(buckets)[v];
    }
    for (uint32_t v = threadIdx.x; v < rows * Q; v += blockDim.x) {
        const uint32_t r = quotient(v, Q, recip), q = v - r * Q;
        // (of the rows beside a tile only colour 1: their colour 0 is another workgroup's)
        if (CUTS || (r != 0 && r + 1 != rows)) *in_lds(0, r, q) = *in_mem(0, r, q);
        *in_lds(1, r, q) = *in_mem(1, r, q);
    }
    const auto bounds = [&](uint32_t s, uint32_t& lo, uint32_t& hi) {
        lo = CUTS ? k - s : 1 + s;
        hi = CUTS ? k + s : rows - 1 - s;
    };
    // proposals: two half-sweeps' rows after the planes
    uint32_t* props = reinterpret_cast<uint32_t*>(B);
    const uint32_t nb = row_blocks(Q), s_first = CUTS ? 1 : 0;
    uint32_t lo, hi;
    bounds(s_first, lo, hi);
    if (MODEL == 1 && WORDS)
        draw_proposals(props + (s_first & 1u) * rows * nb * 4, lo, hi, first, L, Q, s_first & 1u, t, k0, k1);
    __syncthreads();
    const Rule rule{k0, k1, T4, MODEL == 2 ? lt.T[8] : T8, tabs.bc.e, B, tabs.lut, lt.kmax};
    for (uint32_t s = s_first; s < k; ++s) {
        const uint32_t c = s & 1u;
        bounds(s, lo, hi);
        const uint32_t U = WORDS ? W : Q;
        for (uint32_t v = threadIdx.x; v < (hi - lo) * U; v += blockDim.x) {
            const uint32_t dr = quotient(v, U, WORDS ? recip_w : recip), r = lo + dr, w = v - dr * U;
            char* own = lds + (c * rows + r) * rowB;
            const char* oth = lds + ((1 - c) * rows + r) * rowB;
            const uint32_t y = row_of(first, r, L);
            if (WORDS)
                update_word<MODEL>(rule, own, oth - rowB, oth, oth + rowB, w, W, y, L, c, t + (s >> 1), [&](uint32_t kv) {
                    return proposal_word(props + (c * rows + r) * nb * 4, kv, y, Q);
                });
            else
                update_vector<MODEL>(rule, own, oth - rowB, oth, oth + rowB, w, Q, y, L, c, t + (s >> 1));
        }
        if (MODEL == 1 && WORDS && s + 1 < k) {
            bounds(s + 1, lo, hi);
            draw_proposals(props + (1 - c) * rows * nb * 4, lo, hi, first, L, Q, 1 - c, t + ((s + 1) >> 1), k0, k1);
        }
        __syncthreads();
    }
    // what this workgroup changed: colour c from its first half-sweep on
    const uint32_t lo0 = CUTS ? k - (k - 2) : 1, hi0 = CUTS ? k + (k - 2) : rows - 1;
    const uint32_t lo1 = CUTS ? 1 : 2, hi1 = CUTS ? 2 * k - 1 : rows - 2;
    for (uint32_t v = threadIdx.x; v < rows * Q; v += blockDim.x) {
        const uint32_t r = quotient(v, Q, recip), q = v - r * Q;
        if (r >= lo0 && r < hi0) *in_mem(0, r, q) = *in_lds(0, r, q);
        if (r >= lo1 && r < hi1) *in_mem(1, r, q) = *in_lds(1, r, q);
    }
}

// ---------------------------------------------------------------------------
// One half-sweep of a small lattice, a thread per word: a thread's chain is a
// quarter of a vector's and there are four times the waves, without the two
// row steps of a band.  1-bit cells take the exact search, so that a single
// sweep needs no bucket table.  One sweep in us, against the band kernels
// (launching takes about 3.7 of each half): Ising L = 256 7.7 against 8.6, 2048
// 7.9 against 9.6; Blume-Capel 8.0 against 12.6 and 9.9 against 13.6; 1-bit 7.0
// against 22.2 and 7.5 against 27.4.
// ---------------------------------------------------------------------------
template <int MODEL>
__global__ __launch_bounds__(256) void half_words_kernel(uint32_t* __restrict__ planes, uint32_t L, uint32_t c, uint32_t t,
                                                         uint32_t k0, uint32_t k1, uint32_t T4, uint32_t T8, BCTable bc,
                                                         LutTable lt)
{
    constexpr int CB = MODEL == 2 ? 1 : 4;
    __shared__ ResidentLds tabs;
    const uint32_t rowB = (L >> 4) * CB, W = rowB >> 2;
    if (MODEL == 1) dev::load_bc_table(tabs.bc, bc);
    if (MODEL == 2) {
        if (threadIdx.x < 16) tabs.lut[threadIdx.x] = lt.T[threadIdx.x];
        __syncthreads();
    }
    const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= L * W) return;
    const uint32_t y = quotient(g, W, reciprocal(W)), w = g - y * W;
    char* own = reinterpret_cast<char*>(planes) + (size_t)c * L * rowB + (size_t)y * rowB;
    const char* oth = reinterpret_cast<const char*>(planes) + (size_t)(1 - c) * L * rowB;
    const Rule rule{k0, k1, T4, MODEL == 2 ? lt.T[8] : T8, tabs.bc.e, nullptr, tabs.lut, lt.kmax};
    update_word<MODEL, true>(rule, own, oth + (size_t)(y == 0 ? L - 1 : y - 1) * rowB, oth + (size_t)y * rowB,
                             oth + (size_t)(y + 1 == L ? 0 : y + 1) * rowB, w, W, y, L, c, t, [&](uint32_t kv) {
                                 const Philox4 p = philox4x32_10(kv >> 7, 0u, t, 2u + c, k0, k1);
                                 return philox_word(p, (int)((kv >> 5) & 3));
                             });
}

// No more threads than a plane has 16-byte vectors, in whole waves.
uint32_t threads_of(int64_t vectors, int64_t most)
{
    return (uint32_t)std::max<int64_t>(64, std::min<int64_t>(most, (vectors + 63) / 64 * 64));
}

template <class K, class... A>
hipError_t go(K kernel, uint32_t grid, uint32_t threads, size_t lds, hipStream_t s, A... args)
{
    const hipError_t e = allow_lds(kernel, lds, kMostLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, s, args...);
    return hipGetLastError();
}

}  // namespace

// Tiles of k half-sweeps: as many as have at least 2 k rows, but no more than
// compute units (512 tiles at L = 5120: 24.5 us a sweep, 256: 16.4).
static int64_t trapezoid_tiles(int64_t L, int64_t k) { return std::max<int64_t>(1, std::min<int64_t>(L / (2 * k), 256)); }

// Word by word (1-bit cells, and 4-bit ones below L = 4096), or vectors: at
// L = 3008 10.1 against 10.5 us a sweep (Blume-Capel 12.4, 14.1), at L = 5120
// 18.2 against 16.4 (22.2, 20.6); 1-bit L = 4096 8.7 against 17.2.
static bool trapezoid_words(const Geom& g) { return g.cb == 1 || g.L < 4096; }

static size_t trapezoid_lds(const Geom& g, int64_t k)
{
    const int64_t tiles = trapezoid_tiles(g.L, k);
    const int64_t rows = std::max<int64_t>((g.L + tiles - 1) / tiles + 2, 2 * k);
    // (and room for the buckets or proposals)
    const size_t extra = g.cb == 1 ? (size_t)kLutBucketBytes
                         : trapezoid_words(g) ? (size_t)(2 * rows * row_blocks((uint32_t)g.Q) * 16) : 0;
    return (size_t)(2 * rows * g.Q * 16) + extra;
}

// Sizes at which the workgroups of a launch per half-sweep (2-row bands, 256
// threads) just fill two or four rounds of the compute units, so that it is at
// its best: 1 where only runs of two sweeps lose to it (time of two sweeps, and
// five, against it: 4-bit L = 3904 .. 4096 1.00 .. 1.03, 0.96 .. 0.99; 1-bit
// L = 11264 1.02, 1.00), 2 where all do (1-bit L = 11520 1.05, 1.04, four sweeps
// 1.00), else 0 (L = 3840 0.97, 4160 0.86; 11008 0.98, 11776 0.84).
static int full_rounds(const Geom& g)
{
    if (g.cb == 4) return g.L >= 3904 && g.L <= 4096 ? 1 : 0;
    return g.L > 11264 && g.L <= 11520 ? 2 : g.L > 11008 && g.L <= 11264 ? 1 : 0;
}

int64_t trapezoid_least(const Geom& g) { return full_rounds(g) ? 3 : 2; }

int64_t trapezoid_sweeps(const Geom& g)
{
    if (g.L < 128 || g.L > (g.cb == 1 ? kTrapezoidMaxLutL : kTrapezoidMaxL) || full_rounds(g) == 2) return 0;
    // Four: fewer launches.  Three have more tiles, L / 12 against L / 16, for the
    // compute units, which 4-bit words gain from in between: us a sweep at 24
    // sweeps, three against four, L = 1024 5.1 against 4.9, 1408 5.8 / 5.9, 1536
    // 5.8 / 6.1 (Blume-Capel 7.2 / 7.7), 3008 9.1 / 9.8, 3584 10.8 / 11.2; 3648
    // 11.5 / 11.6, where four sweeps take four in one run and three do not,
    // 3904 12.6 / 12.4.  Two are nowhere better than three by more than 5% (L =
    // 2048 6.6, 6.7), six at L <= 384 and from 6144 on, by up to 8% and 3%.
    const int64_t m = g.cb == 4 && g.L >= 1536 && g.L <= 3584 ? 3 : 4;
    return trapezoid_lds(g, 2 * m) <= kMostLds ? m : 0;
}

hipError_t launch_trapezoids(const Geom& g, int model, int64_t sweeps, uint32_t t, uint64_t seed,
                             uint32_t T4, uint32_t T8, const BCTable& bc, const LutTable& lt, const void* buckets,
                             hipStream_t s)
{
    const int64_t k = 2 * sweeps;
    if (sweeps < 2 || sweeps > trapezoid_sweeps(g)) return hipErrorInvalidValue;
    const uint32_t tiles = (uint32_t)trapezoid_tiles(g.L, k);
    const size_t lds = trapezoid_lds(g, k);
    const bool words = trapezoid_words(g);
    const uint32_t threads = threads_of((g.L + tiles - 1) / tiles * g.Q * (words ? 4 : 1), kMaxThreads);
    const auto both = [&](auto tile, auto cut) {
        hipError_t e = hipSuccess;
        for (int cuts = 0; cuts < 2 && e == hipSuccess; ++cuts)
            e = go(cuts ? cut : tile, tiles, threads, lds, s, g.plane0, (uint32_t)g.L, tiles, (uint32_t)k, t,
                   (uint32_t)seed, (uint32_t)(seed >> 32), T4, T8, bc, lt, reinterpret_cast<const uint2*>(buckets));
        return e;
    };
    if (model == 2) return both(trapezoid_kernel<2, true, false>, trapezoid_kernel<2, true, true>);
    if (model == 1)
        return words ? both(trapezoid_kernel<1, true, false>, trapezoid_kernel<1, true, true>)
                     : both(trapezoid_kernel<1, false, false>, trapezoid_kernel<1, false, true>);
    return words ? both(trapezoid_kernel<0, true, false>, trapezoid_kernel<0, true, true>)
                 : both(trapezoid_kernel<0, false, false>, trapezoid_kernel<0, false, true>);
}

bool half_by_words(const Geom& g) { return g.L <= (g.cb == 1 ? kHalfWordsMaxLutL : kHalfWordsMaxL); }

hipError_t launch_half_words(const Geom& g, int model, int color, uint32_t t, uint64_t seed, uint32_t T4, uint32_t T8,
                             const BCTable& bc, const LutTable& lt, hipStream_t s)
{
    if (!half_by_words(g)) return hipErrorInvalidValue;
    const uint32_t grid = (uint32_t)((g.plane_words() + 255) / 256);
    const auto run = [&](auto kernel) {
        return go(kernel, grid, 256, 0, s, g.plane0, (uint32_t)g.L, (uint32_t)color, t, (uint32_t)seed,
                  (uint32_t)(seed >> 32), T4, T8, bc, lt);
    };
    return model == 0 ? run(half_words_kernel<0>) : model == 1 ? run(half_words_kernel<1>) : run(half_words_kernel<2>);
}

hipError_t launch_resident(const GroupDesc& d, uint32_t n, const BCTable& bc, const LutTable& lt, hipStream_t s)
{
    const int model = (int)d.model;
    const int64_t L = d.L, words = L * L / (model == 2 ? 64 : 16);
    const size_t props = model == 1 ? (size_t)(2 * L * row_blocks((uint32_t)(L >> 6)) * 16) : 0;
    const size_t lds = resident_lds(model, L) + props;
    const uint32_t threads = threads_of(words, kMaxThreads);
    const auto run = [&](auto kernel) { return go(kernel, 1, threads, lds, s, d, n, bc, lt); };
    return model == 0 ? run(resident_kernel<0>) : model == 1 ? run(resident_kernel<1>) : run(resident_kernel<2>);
}

hipError_t launch_group_resident(const GroupDesc* desc, int count, size_t lds, int64_t vectors, uint32_t s0, uint32_t s1,
                                 const uint2* bc_tables, const LutRec* luts, hipStream_t s)
{
    const uint32_t threads = threads_of(vectors, count > 256 && lds <= 76u * 1024u ? 512 : kMaxThreads);
    return go(group_resident_kernel, (uint32_t)count, threads, lds, s, desc, s0, s1, bc_tables, luts);
}

}  // namespace mcl
