// ne_sub_device.hpp -- device code of the North-East model by the paper's
// random sub-lattice algorithm (Sec. 3.2) for gfx950; kernels_ne_sub_b*.hip
// instantiate it for one sub-lattice side each (separate translation units
// compile in parallel).
//
// The lattice is cut into Q square sub-lattices of B x B sites.  One launch
// processes every sub-lattice once: q = B^2 / (2 lambda) iterations, each of
// which draws lambda random sites of the sub-lattice and updates them
// together; two launches make a sweep.  Neighbours in other sub-lattices (the
// north row and east column) are read as they were when the launch started:
// the launch reads one copy of the lattice and writes the other.  Neighbours
// in the same sub-lattice are read as they were at the start of the iteration.
//
// Balanced variant (end of Sec. 3.2): each iteration draws lambda sites of
// colour 0, then lambda sites of colour 1 (half h); P/(8 lambda) iterations per
// launch, four launches per sweep.  Sites of one colour are not neighbours, so
// the attempts of a half only read frozen neighbours; when attempts of a half
// draw the same site only the lowest-numbered one applies.
//
// Mapping: a sub-lattice belongs to one wavefront, lambda/2 lanes of it, each
// lane making two attempts per step (an iteration, or a half of one) from one
// Philox4x32-10 call (counter (tau, a/2, launch, 2) for attempts a, a+1; tag 3
// when balanced).  Because a whole sub-lattice lives in one wavefront, a step
// needs no barrier: the wavefront's LDS instructions execute in program order,
// so every read of a step precedes every write of it.  A workgroup is one
// wavefront holding up to 64/(lambda/2) sub-lattices in LDS.
//
// What bounds it: instructions.  At L = 4096, B = 32, lambda = 16 the algorithm
// leaves 2 waves per SIMD, all resident at once, so a launch is the sum of its
// phases: 4.5 us to start, load and store, 11 us for 32 steps, of which the draws
// are 4.7.  Hence as little as possible around a draw:
// - LDS holds each sub-lattice as one bit row per lattice row (the occupations;
//   the north row first), so an attempt's site and its north and east neighbours
//   are two rows read by one instruction and 12 instructions decide it (B = 64,
//   whose rows are two words: 18).  The rows of two steps are read together; the
//   second's again only if an attempt of the wavefront was accepted in the first.
//   (Four steps together 16.0 us a launch, two 15.7.  Deciding four steps from the
//   same rows and again after an accepted one: 20.0 us against 18.8 then.)
// - Accepted moves are kept as lane masks, so the test whether there are any is
//   scalar (as bools: 18.3 us a launch).
// - Between the launches of one call the lattice is kept as those bit rows, an
//   eighth of the bytes for the occupations and as much for the flags: 8 MB
//   instead of 33 MB a launch, and nothing to repack.  The call's first launch
//   reads colour arrays, its last one writes them.  (Colour arrays at every
//   launch: 24 us.)
// Before, with bytes in LDS and memory and three byte reads per attempt: 22.2 us.
//
// Accepted moves clear or set the site's bit with LDS atomics (AND for a
// down-flip, OR for an up-flip; both are issued, one of them with nothing to
// do, and nothing waits until the last) and set its "has flipped" flag in a
// second bit row.  Attempts of one step on one site all see the same n, so the
// value an atomic returns tells whether another attempt already changed the site:
// each changed site is counted once, and a site drawn twice flips once.  The
// balanced variant keeps an owner word per site of a colour for the steps with
// accepted moves: attempts post their number with an LDS atomic minimum, read it
// back, and only the owner may apply its move, by XOR.
//
// Records: the first launch of a sweep also measures the lattice it starts
// from -- the state after the previous sweep -- from the sub-lattices it has
// just loaded (bonds to the north and east neighbours, which tile the lattice's
// bonds exactly once), so no separate pass reads the lattice for that record.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "philox.hpp"
#include "site_update.hpp"
#include "spinlat_internal.h"

namespace spinlat {

namespace nesub {

// Bytes of LDS per one-wavefront workgroup, while a CU has one workgroup at most,
// and for more of them (owner words make the difference, balanced us per sweep at c =
// 0.1, 33 against 19 kB: B = 64, lambda = 16: L = 1536 128 and 163, L = 4096 232 and
// 147).
constexpr int kLdsBudget = 32768, kLdsBudgetShared = 19000;
constexpr uint32_t kTagNeSub = 2u;
constexpr uint32_t kTagNeBal = 3u;

constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v / 2); }

// ---- bit rows --------------------------------------------------------------
// Row: a row in LDS and registers; Bits: a row, or a column, between launches.
template <int B>
struct BitRows;
template <>
struct BitRows<8> {
    using Row = uint32_t;
    using Bits = uint8_t;
};
template <>
struct BitRows<16> {
    using Row = uint32_t;
    using Bits = uint16_t;
};
template <>
struct BitRows<32> {
    using Row = uint32_t;
    using Bits = uint32_t;
};
template <>
struct BitRows<64> {
    using Row = unsigned long long;
    using Bits = unsigned long long;
};

// LDS of one sub-lattice: rows[0] the north row, rows[1 ..] its own, their
// flags, and (B >= 32) the east column.  For B < 32 the east neighbour of a
// row's last site is bit B of the row.
// Words of 32 bits, which attempts read and change: a row of B = 64 is two.
template <int B>
struct alignas(8) BitTile {
    static constexpr int W = B == 64 ? 2 : 1;
    uint32_t rows[W * (B + 1)], flags[W * B], ecol[W];
};

template <int B>
__device__ __forceinline__ typename BitRows<B>::Row row_of(const uint32_t* words, uint32_t r)
{
    if constexpr (B == 64) return words[2 * r] | (unsigned long long)words[2 * r + 1] << 32;
    else return words[r];
}

template <int B>
__device__ __forceinline__ void set_row(uint32_t* words, uint32_t r, typename BitRows<B>::Row v)
{
    if constexpr (B == 64) {
        words[2 * r] = (uint32_t)v;
        words[2 * r + 1] = (uint32_t)(v >> 32);
    } else {
        words[r] = v;
    }
}

template <int B>
__device__ __forceinline__ void or_row(uint32_t* words, typename BitRows<B>::Row v)
{
    atomicOr(words, (uint32_t)v);
    if constexpr (B == 64) atomicOr(words + 1, (uint32_t)(v >> 32));
}

// Whether the lanes of a sub-lattice put a column together by ballots, one per row
// of a lane (few, then), or by LDS atomics.  Where a wavefront holds one sub-lattice,
// the compiler makes an atomic on its column a loop over the lanes: 1.4 us a launch of
// lambda = 128 (us per sweep: B = 16, L = 16 9.5, with ballots 6.3; B = 64, L = 256 23.1 and
// 15.7).
template <int LPT>
constexpr bool column_by_ballot()
{
    return LPT >= 16;
}

// bit of every lane of this lane's sub-lattice, lane l's at bit l
template <int LPT>
__device__ __forceinline__ uint64_t group_ballot(bool bit)
{
    const uint64_t m = __builtin_amdgcn_ballot_w64(bit);
    if constexpr (LPT == 64) return m;
    else return (m >> (threadIdx.x / LPT * LPT)) & ((1ull << LPT) - 1u);
}

template <int B, bool BAL>
constexpr int owner_words()
{
    return BAL ? B * B / 2 : 0;
}

template <int B, int LPT, bool BAL>
constexpr int tiles_per_wave(int budget)
{
    const int fit = budget / ((int)sizeof(BitTile<B>) + 4 * owner_words<B, BAL>());
    return 64 / LPT < fit ? 64 / LPT : fit;
}

// The lattice between launches, in the colour arrays' memory: occupations as
// Bits[sub-lattice][row] in colour 0's; in colour 1's the flags likewise, then
// each sub-lattice's first column.  B / 8 bytes a row of B / 2 per colour.
template <int B>
struct BitLattice {
    using Bits = typename BitRows<B>::Bits;
    Bits *rows, *flags, *column;
    __device__ __forceinline__ BitLattice(uint8_t* c0, uint8_t* c1, uint32_t ntiles)
        : rows(reinterpret_cast<Bits*>(c0)),
          flags(reinterpret_cast<Bits*>(c1)),
          column(reinterpret_cast<Bits*>(c1) + (size_t)ntiles * B)
    {
    }
};

template <int N>
struct ColourVec {
    uint32_t w[N / 4];
};

template <int N>
__device__ __forceinline__ ColourVec<N> load_vec(const uint8_t* p)
{
    ColourVec<N> v;
    if constexpr (N == 16) {
        const uint4 q = *reinterpret_cast<const uint4*>(p);
        v.w[0] = q.x; v.w[1] = q.y; v.w[2] = q.z; v.w[3] = q.w;
    } else if constexpr (N == 8) {
        const uint2 q = *reinterpret_cast<const uint2*>(p);
        v.w[0] = q.x; v.w[1] = q.y;
    } else {
        v.w[0] = *reinterpret_cast<const uint32_t*>(p);
    }
    return v;
}

template <int N>
__device__ __forceinline__ void store_vec(uint8_t* p, const ColourVec<N>& v)
{
    if constexpr (N == 16) {
        *reinterpret_cast<uint4*>(p) = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
    } else if constexpr (N == 8) {
        *reinterpret_cast<uint2*>(p) = make_uint2(v.w[0], v.w[1]);
    } else {
        *reinterpret_cast<uint32_t*>(p) = v.w[0];
    }
}

// A lane's rows in steps of up to 64 registers of loads in flight.
template <int B, int LPT>
struct RowSteps {
    static constexpr int most = B <= 32 ? 8 : 4;
    static constexpr int rows = (B + LPT) / LPT;  // of B + 1, per lane
    static constexpr int steps = (rows + most - 1) / most;
    static constexpr int per_step = (rows + steps - 1) / steps;
};

// Bit k of each byte of e (4 sites at even x) and o (odd x), in x order: the
// result's bits k .. k + 7.
template <int K>
__device__ __forceinline__ uint32_t gather8(uint32_t e, uint32_t o)
{
    const uint32_t lo = __builtin_amdgcn_udot4(o & (0x01010101u << K), 0x80200802u, 0u, false);
    return __builtin_amdgcn_udot4(e & (0x01010101u << K), 0x40100401u, lo, false);
}

// Bits 0, 2, 4, 6 of v to bit 0 of bytes 0 .. 3 (the products' other terms meet
// in bits that no byte starts at).
__device__ __forceinline__ uint32_t spread4(uint32_t v)
{
    return __umul24(v & 0x55u, 0x41041u) & 0x01010101u;
}

// Sub-lattice (x0, y0) of the colour arrays into bit rows; lanes l of LPT share it.
template <int B, int LPT>
__device__ __forceinline__ void load_colours(const NeSubArgs& a, BitTile<B>& t, uint32_t l, uint32_t x0, uint32_t y0)
{
    using Row = typename BitRows<B>::Row;
    using Steps = RowSteps<B, LPT>;
    constexpr int UNIT = B / 2 < 16 ? B / 2 : 16;  // bytes of a colour vector load
    constexpr int NV = B / 2 / UNIT;
    constexpr int K = Steps::per_step;
    const uint32_t xe = x0 + B == a.L ? 0u : x0 + B;
    constexpr bool BALLOT = column_by_ballot<LPT>();
    if (B >= 32 && !BALLOT && l == 0) set_row<B>(t.ecol, 0, 0);
    Row ecol = 0;
#pragma nounroll
    for (int s = 0; s < Steps::steps; ++s) {
        ColourVec<UNIT> e[K][NV], o[K][NV];
        uint32_t east[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t pr = min(l + (uint32_t)((s * K + i) * LPT), (uint32_t)B);
            const uint32_t y = pr == 0 ? (y0 == 0 ? a.L - 1 : y0 - 1) : y0 + pr - 1u;
            const size_t off = (size_t)y * a.Lh;
            // colour 1 holds the even x of odd rows
            const uint8_t* even = ((y & 1u) != 0 ? a.src[1] : a.src[0]) + off + (x0 >> 1);
            const uint8_t* odd = ((y & 1u) != 0 ? a.src[0] : a.src[1]) + off + (x0 >> 1);
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                e[i][u] = load_vec<UNIT>(even + u * UNIT);
                o[i][u] = load_vec<UNIT>(odd + u * UNIT);
            }
            // east neighbour of the row's last site: colour (x0 + B + y) & 1
            east[i] = a.src[(xe + y) & 1u][off + (xe >> 1)];
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t pr = l + (uint32_t)((s * K + i) * LPT);
            Row row = 0, flags = 0;
#pragma unroll
            for (int u = 0; u < NV; ++u)
#pragma unroll
                for (int k = 0; k < UNIT / 4; ++k) {
                    const int sh = 8 * (u * (UNIT / 4) + k);
                    row |= (Row)gather8<0>(e[i][u].w[k], o[i][u].w[k]) << sh;
                    flags |= (Row)(gather8<1>(e[i][u].w[k], o[i][u].w[k]) >> 1) << sh;
                }
            if (B < 32) row |= (Row)(east[i] & 1u) << (B & 31);
            if (pr <= (uint32_t)B) set_row<B>(t.rows, pr, row);
            const bool own = pr - 1u < (uint32_t)B;
            if (own) set_row<B>(t.flags, pr - 1u, flags);
            if constexpr (B >= 32 && BALLOT) {
                const uint64_t m = group_ballot<LPT>(own && (east[i] & 1u) != 0);
                const uint32_t first = (uint32_t)((s * K + i) * LPT);  // pr of lane 0
                ecol |= first == 0 ? (Row)(m >> 1) : (Row)m << min(first - 1u, (uint32_t)(B - 1));
            } else if (B >= 32 && own) {
                ecol |= (Row)(east[i] & 1u) << (pr - 1u);
            }
        }
    }
    if constexpr (B >= 32 && BALLOT) {
        if (l == 0) set_row<B>(t.ecol, 0, ecol);
    } else if constexpr (B >= 32) {
        or_row<B>(t.ecol, ecol);
    }
}

// Sub-lattice (tx, ty) of bit rows.
template <int B, int LPT>
__device__ __forceinline__ void load_bits(const NeSubArgs& a, BitTile<B>& t, uint32_t l, uint32_t tx, uint32_t ty)
{
    using Row = typename BitRows<B>::Row;
    using Bits = typename BitRows<B>::Bits;
    constexpr int R = (B + LPT - 1) / LPT;
    constexpr int K = R < 8 ? R : 8;  // rows in flight
    const BitLattice<B> src(const_cast<uint8_t*>(a.src[0]), const_cast<uint8_t*>(a.src[1]), a.ntiles);
    const uint32_t tau = ty * a.tiles_x + tx;
    const uint32_t north = (ty == 0 ? a.tiles_x - 1 : ty - 1) * a.tiles_x + tx;
    const uint32_t east = ty * a.tiles_x + (tx + 1 == a.tiles_x ? 0u : tx + 1);
    const Bits column = src.column[east];
    const Row above = src.rows[(size_t)north * B + (B - 1)];
#pragma nounroll
    for (int i0 = 0; i0 < R; i0 += K) {
        Bits row[K], flags[K];
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t r = min(l + (uint32_t)((i0 + i) * LPT), (uint32_t)(B - 1));
            row[i] = src.rows[(size_t)tau * B + r];
            flags[i] = src.flags[(size_t)tau * B + r];
        }
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t r = l + (uint32_t)((i0 + i) * LPT);
            if (r < (uint32_t)B) {
                set_row<B>(t.rows, r + 1, B < 32 ? (Row)row[i] | (((Row)column >> r) & 1u) << (B & 31) : (Row)row[i]);
                set_row<B>(t.flags, r, flags[i]);
            }
        }
    }
    if (l == 0) {
        set_row<B>(t.rows, 0, above);
        set_row<B>(t.ecol, 0, column);
    }
}

// Occupation, bonds to the north and east neighbours, and sites with the flag
// clear, of the rows as loaded.
template <int B, int LPT>
__device__ __forceinline__ void observe_rows(const BitTile<B>& t, uint32_t l, int& mag, int& bond, int& fresh)
{
    using Row = typename BitRows<B>::Row;
    constexpr Row mask = B >= 32 ? ~(Row)0 : ((Row)1 << (B & 31)) - 1;
    for (int r = (int)l; r < B; r += LPT) {
        const Row row = row_of<B>(t.rows, r + 1), n = row & mask;
        Row east = row >> 1;
        if (B >= 32) east |= ((row_of<B>(t.ecol, 0) >> r) & 1u) << (B - 1);
        mag += __builtin_popcountll(n);
        bond += __builtin_popcountll(n & row_of<B>(t.rows, r)) + __builtin_popcountll(n & east);
        fresh += B - __builtin_popcountll(row_of<B>(t.flags, r));
    }
}

// The rows to the colour arrays of the destination copy.
template <int B, int LPT>
__device__ __forceinline__ void store_colours(const NeSubArgs& a, const BitTile<B>& t, uint32_t l, uint32_t x0, uint32_t y0)
{
    using Row = typename BitRows<B>::Row;
    constexpr int UNIT = B / 2 < 16 ? B / 2 : 16;
#pragma unroll 2
    for (uint32_t r = l; r < (uint32_t)B; r += LPT) {
        const Row row = row_of<B>(t.rows, r + 1), flags = row_of<B>(t.flags, r);
        const size_t off = (size_t)(y0 + r) * a.Lh + (x0 >> 1);
        // y0 is even; colour 1 holds the even x of odd rows
        uint8_t* even = ((r & 1u) != 0 ? a.dst[1] : a.dst[0]) + off;
        uint8_t* odd = ((r & 1u) != 0 ? a.dst[0] : a.dst[1]) + off;
#pragma unroll
        for (int u = 0; u < B / 2 / UNIT; ++u) {
            ColourVec<UNIT> e, o;
#pragma unroll
            for (int k = 0; k < UNIT / 4; ++k) {
                const int sh = 8 * (u * (UNIT / 4) + k);
                const uint32_t n8 = (uint32_t)(row >> sh), f8 = (uint32_t)(flags >> sh);
                e.w[k] = spread4(n8) | (spread4(f8) << 1);
                o.w[k] = spread4(n8 >> 1) | (spread4(f8 >> 1) << 1);
            }
            store_vec<UNIT>(even + u * UNIT, e);
            store_vec<UNIT>(odd + u * UNIT, o);
        }
    }
}

// The rows as bit rows.
template <int B, int LPT>
__device__ __forceinline__ void store_bits(const NeSubArgs& a, BitTile<B>& t, uint32_t l, uint32_t tau)
{
    using Row = typename BitRows<B>::Row;
    using Bits = typename BitRows<B>::Bits;
    constexpr bool BALLOT = column_by_ballot<LPT>();
    const BitLattice<B> dst(a.dst[0], a.dst[1], a.ntiles);
    if (!BALLOT && l == 0) set_row<B>(t.ecol, 0, 0);
    Row column = 0;
    constexpr int R = (B + LPT - 1) / LPT;  // rows of a lane; LPT > B: of the first B lanes
#pragma unroll 4
    for (int i = 0; i < R; ++i) {
        const uint32_t r = l + (uint32_t)(i * LPT);
        const bool own = LPT <= B || r < (uint32_t)B;
        const Row row = row_of<B>(t.rows, (own ? r : 0u) + 1u);
        if (own) {
            dst.rows[(size_t)tau * B + r] = (Bits)row;
            dst.flags[(size_t)tau * B + r] = (Bits)row_of<B>(t.flags, r);
        }
        if constexpr (BALLOT) column |= (Row)group_ballot<LPT>(own && (row & 1u) != 0) << (i * LPT);
        else column |= (row & 1u) << r;
    }
    if constexpr (!BALLOT) {
        or_row<B>(t.ecol, column);
        asm volatile("" ::: "memory");  // all lanes' parts
        column = row_of<B>(t.ecol, 0);
    }
    if (l == 0) dst.column[tau] = (Bits)column;
}

// Wavefront sums of the per-lane counts into the records: one atomic
// instruction, four lanes on one line or two (an instruction each: 1.1 us more
// per launch of 2048 waves, which meet on kSub lines).
__device__ __forceinline__ void add_counts(const NeSubArgs& a, uint32_t lane, int changed, int mag,
                                           int bond, int fresh)
{
    int sum = wave_sum(changed);
    unsigned long long* p = a.acc + 2;
    if (a.obs) {
        const int q[3] = {wave_sum(bond), wave_sum(mag), wave_sum(fresh)};
        if (lane != 2) {
            sum = lane == 0 ? q[0] : lane == 1 ? q[1] : q[2];
            p = a.obs + lane;
        }
    }
    if ((lane == 2 || (a.obs && lane < 4)) && sum != 0)
        atomicAdd(p + (blockIdx.x % kSub) * kSubStride, (unsigned long long)sum);
}

// The site an attempt's word draws: row r, column c() (c5: with other bits above
// the low 5, which a shift by it ignores).  Balanced: a site of colour h.
template <int B, bool BAL>
struct Draw {
    uint32_t r, c5;
    __device__ __forceinline__ Draw(uint32_t word, int h)
        : r(word >> (32 - ilog2(B))),
          c5(BAL ? 2u * (word >> (33 - 2 * ilog2(B))) + ((r + (uint32_t)h) & 1u) : word >> (32 - 2 * ilog2(B)))
    {
    }
    __device__ __forceinline__ uint32_t c() const { return c5 & (B - 1); }
};

// The rows an attempt reads, its own and the one to the north.
template <int B>
struct RowPair {
    uint32_t north[BitTile<B>::W], own[BitTile<B>::W];
};

template <int B, bool WRAP>
__device__ __forceinline__ RowPair<B> read_rows(const BitTile<B>& t, uint32_t word)
{
    constexpr uint32_t W = BitTile<B>::W;
    const uint32_t r = word >> (32 - ilog2(B));
    RowPair<B> p;
    // one sub-lattice: the periodic neighbours are inside it
    const uint32_t* north = t.rows + W * (WRAP && r == 0 ? (uint32_t)B : r);
    __builtin_memcpy(p.north, __builtin_assume_aligned(north, 4 * W), 4 * W);
    __builtin_memcpy(p.own, __builtin_assume_aligned(t.rows + W * (r + 1), 4 * W), 4 * W);
    return p;
}

// Balanced: whether each attempt is the lowest-numbered one on its site in this
// half; owner words are as before again afterwards.
template <int B>
__device__ __forceinline__ void claim(uint32_t* owner, uint32_t l, const Words4& w, bool (&win)[2])
{
    uint32_t idx[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        idx[m] = w.w[2 * m] >> (33 - 2 * ilog2(B));
        atomicMin(owner + idx[m], 2u * l + (uint32_t)m);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
        win[m] = __hip_atomic_load(owner + idx[m], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == 2u * l + (uint32_t)m;
    asm volatile("" ::: "memory");  // all lanes have read
#pragma unroll
    for (int m = 0; m < 2; ++m) owner[idx[m]] = 0xFFFFFFFFu;
}

template <int B, int LPT, bool WRAP, bool BAL, int TPW>
__global__ void __launch_bounds__(64) k_ne_sub(NeSubArgs a)
{
    static_assert(TPW >= 1, "a sub-lattice must fit the LDS budget");
    constexpr uint32_t TAG = BAL ? kTagNeBal : kTagNeSub;
    constexpr int STEPS = ne_sub_steps(B, 2 * LPT, BAL);
    // steps whose rows are read together: few wavefronts with many steps each have
    // the latency of a step as their bound (B = 64, L = 512 two against four, us per
    // sweep: lambda = 16 77.5 and 73.4, lambda = 32 41.2 and 43.1)
    constexpr int G = STEPS < 2 ? 1 : B == 64 && LPT <= 8 ? 4 : 2;
    constexpr int OW = owner_words<B, BAL>();
    __shared__ BitTile<B> lds[TPW];
    __shared__ uint32_t lds_owner[BAL ? TPW * OW : 1];

    const uint32_t lane = threadIdx.x;
    const uint32_t g = lane / LPT;
    const uint32_t l = lane % LPT;
    const uint32_t tau = blockIdx.x * TPW + g;
    int changed = 0, mag = 0, bond = 0, fresh = 0;
    if (g < (uint32_t)TPW && tau < a.ntiles) {
        BitTile<B>& t = lds[g];
        uint32_t* owner = lds_owner + (BAL ? g * OW : 0);
        const uint32_t tx = tau % a.tiles_x, ty = tau / a.tiles_x;
        if (a.bits_in)
            load_bits<B, LPT>(a, t, l, tx, ty);
        else
            load_colours<B, LPT>(a, t, l, tx * B, ty * B);
        if (BAL)
            for (int i = (int)l; i < OW; i += LPT) owner[i] = 0xFFFFFFFFu;
        asm volatile("" ::: "memory");  // other lanes' rows from here on
        if (a.obs) observe_rows<B, LPT>(t, l, mag, bond, fresh);
        const uint32_t ecol_lo = B >= 32 && !WRAP ? t.ecol[0] : 0u;
        const uint32_t ecol_hi = B == 64 && !WRAP ? t.ecol[BitTile<B>::W - 1] : 0u;
        const uint64_t may_up = (a.never & 1u) == 0u ? ~0ull : 0ull, may_down = (a.never & 2u) == 0u ? ~0ull : 0ull;

        const PhiloxKey ks = philox_schedule(a.key0, a.key1);
        Words4 w[G];
#pragma unroll
        for (int i = 0; i < G; ++i) w[i] = philox4x32_10(tau, (uint32_t)(i * LPT) + l, a.launch, TAG, ks);
#pragma nounroll
        for (uint32_t j = 0; j < a.steps; j += G) {
            RowPair<B> rows[G][2];
#pragma unroll
            for (int i = 0; i < 2 * G; ++i) rows[i / 2][i & 1] = read_rows<B, WRAP>(t, w[i / 2].w[2 * (i & 1)]);
#pragma unroll
            for (int i = 0; i < 2 * G; ++i)  // together, not each before its use
#pragma unroll
                for (int k = 0; k < BitTile<B>::W; ++k)
                    asm volatile("" : "+v"(rows[i / 2][i & 1].own[k]), "+v"(rows[i / 2][i & 1].north[k]));
            Words4 wn[G];
#pragma unroll
            for (int i = 0; i < G; ++i)
                wn[i] = philox4x32_10(tau, (j + (uint32_t)(G + i)) * LPT + l, a.launch, TAG, ks);
#pragma unroll
            for (int i = 0; i < G; ++i) {
                uint64_t up_mask[2], down_mask[2];  // accepted attempts, by lane
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const Draw<B, BAL> d(w[i].w[2 * m], i & 1);
                    // bit 0 of s the site, bit 1 its east neighbour
                    const RowPair<B>& row = rows[i][m];
                    const bool low = B < 64 || (d.c5 & 32u) == 0u;  // B = 64: the row's first word
                    const uint32_t own_lo = row.own[0], own_hi = row.own[BitTile<B>::W - 1];
                    const uint32_t north_lo = row.north[0], north_hi = row.north[BitTile<B>::W - 1];
                    const uint32_t own = low ? own_lo : own_hi;
                    uint32_t s;
                    if constexpr (B < 32) {
                        s = (WRAP ? (own & ((1u << (B & 31)) - 1u)) | (own << (B & 31)) : own) >> d.c();
                    } else if constexpr (B == 32) {
                        s = __builtin_amdgcn_alignbit(WRAP ? own : ecol_lo >> d.r, own, d.c5);
                    } else {
                        const uint32_t past = WRAP ? own_lo : (d.r & 32u ? ecol_hi : ecol_lo) >> (d.r & 31u);
                        const uint32_t next = low ? own_hi : past;
                        s = __builtin_amdgcn_alignbit(next, own, d.c5);
                    }
                    const uint32_t north = __builtin_amdgcn_ubfe(low ? north_lo : north_hi, B >= 32 ? d.c5 : d.c(), 1);
                    const uint32_t k = north << 2 | (s & 3u), word = w[i].w[2 * m + 1];
                    // accept iff word < thr, thr in [0, 2^32]: word <= thr - 1 unless thr = 0
                    up_mask[m] = __builtin_amdgcn_ballot_w64(k == 6u) &
                                 __builtin_amdgcn_ballot_w64(word <= a.thr_m1_up) & may_up;
                    down_mask[m] = __builtin_amdgcn_ballot_w64(k == 7u) &
                                   __builtin_amdgcn_ballot_w64(word <= a.thr_m1_down) & may_down;
                }
                if ((up_mask[0] | up_mask[1] | down_mask[0] | down_mask[1]) != 0ull) {
                    bool up[2], down[2];
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        up[m] = __builtin_amdgcn_inverse_ballot_w64(up_mask[m]);
                        down[m] = __builtin_amdgcn_inverse_ballot_w64(down_mask[m]);
                    }
                    if constexpr (BAL) {
                        bool win[2];
                        claim<B>(owner, l, w[i], win);
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            up[m] = up[m] && win[m];
                            down[m] = down[m] && win[m];
                        }
                    }
                    if (up[0] || down[0] || up[1] || down[1]) {
                        uint32_t and_old[2], or_old[2], bit[2];
#pragma unroll
                        for (int m = 0; m < 2; ++m) {
                            const Draw<B, BAL> d(w[i].w[2 * m], i & 1);
                            const uint32_t half = B == 64 ? (d.c5 >> 5) & 1u : 0u;
                            uint32_t* row = &t.rows[BitTile<B>::W * (d.r + 1) + half];
                            bit[m] = 1u << (B < 32 ? d.c() : d.c5 & 31u);
                            const uint32_t set = up[m] || down[m] ? bit[m] : 0u;
                            if constexpr (BAL) {  // one attempt per site
                                atomicXor(row, set);
                                changed += set != 0u ? 1 : 0;
                            } else {
                                and_old[m] = atomicAnd(row, down[m] ? ~bit[m] : ~0u);
                                or_old[m] = atomicOr(row, up[m] ? bit[m] : 0u);
                            }
                            atomicOr(&t.flags[BitTile<B>::W * d.r + half], set);
                        }
                        // the first change of the site in this step: n still as at its start
                        if constexpr (!BAL) {
#pragma unroll
                            for (int m = 0; m < 2; ++m)
                                changed +=
                                    (down[m] && (and_old[m] & bit[m]) != 0) || (up[m] && (or_old[m] & bit[m]) == 0) ? 1 : 0;
                        }
                    }
                    asm volatile("" ::: "memory");  // also rows that other lanes changed
#pragma unroll
                    for (int k = 2 * (i + 1); k < 2 * G; ++k)
                        rows[k / 2][k & 1] = read_rows<B, WRAP>(t, w[k / 2].w[2 * (k & 1)]);
                }
            }
#pragma unroll
            for (int i = 0; i < G; ++i) w[i] = wn[i];
        }
        asm volatile("" ::: "memory");
        if (a.bits_out)
            store_bits<B, LPT>(a, t, l, tau);
        else
            store_colours<B, LPT>(a, t, l, tx * B, ty * B);
    }
    add_counts(a, lane, changed, mag, bond, fresh);
}

template <int B, int LPT, bool BAL>
hipError_t launch_one(const NeSubArgs& a, hipStream_t s)
{
    constexpr int WIDE = tiles_per_wave<B, LPT, BAL>(kLdsBudget);
    constexpr int SHARED = tiles_per_wave<B, LPT, BAL>(kLdsBudgetShared);
    const uint32_t wide = (a.ntiles + WIDE - 1) / WIDE, shared = (a.ntiles + SHARED - 1) / SHARED;
    if (a.ntiles == 1)
        hipLaunchKernelGGL((k_ne_sub<B, LPT, true, BAL, 1>), dim3(1), dim3(64), 0, s, a);
    else if (wide <= 256)
        hipLaunchKernelGGL((k_ne_sub<B, LPT, false, BAL, WIDE>), dim3(wide), dim3(64), 0, s, a);
    else
        hipLaunchKernelGGL((k_ne_sub<B, LPT, false, BAL, SHARED>), dim3(shared), dim3(64), 0, s, a);
    return hipGetLastError();
}

template <int B, bool BAL>
hipError_t launch_lambda(const NeSubArgs& a, int lambda, hipStream_t s)
{
    switch (lambda) {
        case 2: return launch_one<B, 1, BAL>(a, s);
        case 4: return launch_one<B, 2, BAL>(a, s);
        case 8: return launch_one<B, 4, BAL>(a, s);
        case 16: return launch_one<B, 8, BAL>(a, s);
        case 32: return launch_one<B, 16, BAL>(a, s);
        case 64: return launch_one<B, 32, BAL>(a, s);
        case 128: return launch_one<B, 64, BAL>(a, s);
    }
    return hipErrorInvalidValue;
}

template <int B>
hipError_t launch_side(const NeSubArgs& a, int lambda, bool balanced, hipStream_t s)
{
    return balanced ? launch_lambda<B, true>(a, lambda, s) : launch_lambda<B, false>(a, lambda, s);
}

}  // namespace nesub

}  // namespace spinlat
