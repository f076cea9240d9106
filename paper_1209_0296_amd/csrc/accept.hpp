// accept.hpp -- Metropolis acceptance of the four sites of a word from threshold
// tables in LDS (device code).
//
// Spin-1/2 lattices and the coupled North-East model: a site has at most 16 table numbers (up to 7 neighbour counts for either
// spin), so a table of all pairs is 2 KiB: one 8-byte read gives two sites'
// thresholds, and its address is one v_dot4 of the word of table numbers with
// two byte weights.  Per word that is 2 address instructions and 2 reads
// against 4 and 4 for one site at a time.  Thresholds are kept as thr - 1
// ("accept iff word <= thr - 1"), so every one must be >= 1.
//
// Spin-1 lattices: 52 entries, one read per site.  What a site may change to
// and which table row that takes are byte permutes, by the site's value and
// the top bit of its second random word, of all four sites at once.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "philox.hpp"
#include "spinlat_internal.h"

namespace spinlat {

// Entry (n0, n1) of two sites' table numbers n in 0 .. 15, at byte 8 n0 + 136 n1
// (the 8 bytes beyond 16 entries spread the rows over the LDS banks).
// n = neighbours at -1 + 8 (s == -1) for spin-1/2, neighbours up + 8 n for
// coupled NE.
struct PairLut {
    uint64_t e[16 * 17];
};

// Built by all threads of the block; NE: the coupled NE numbering.
template <bool NE, int DIM>
__device__ __forceinline__ void build_pair_lut(PairLut& lut, const uint64_t* table)
{
    constexpr int z = 2 * DIM;
    for (int t = threadIdx.x; t < 256; t += blockDim.x) {
        uint32_t v[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int n = k ? t >> 4 : t & 15;
            const int m = (n & 7) <= z ? (n & 7) : z;  // 0 .. z
            const bool up = NE ? (n >> 3) == 1 : (n >> 3) == 0;
            const int nsum = NE ? 2 * m - z : z - 2 * m;
            v[k] = (uint32_t)(table[(up ? 0 : 3) * (2 * z + 1) + nsum + z] - 1ull);
        }
        lut.e[(t & 15) + 17 * (t >> 4)] = (uint64_t)v[0] | ((uint64_t)v[1] << 32);
    }
}

// v_dot4: c + the sum of the four byte products
__device__ __forceinline__ uint32_t udot4(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_udot4(a, b, c, false);
}
__device__ __forceinline__ int32_t sdot4(uint32_t a, uint32_t b, int32_t c)
{
    return __builtin_amdgcn_sdot4((int)a, (int)b, c, false);
}

// Byte mask (that of val per accepted site) of four sites whose table numbers,
// scaled so that byte weights W0 and W1 give the PairLut offset, are in idx.
// `between` runs after the table reads are issued and before their results
// are used.
template <uint32_t W0, uint32_t W1, class F>
__device__ __forceinline__ uint32_t pair_accept(const PairLut& lut, uint32_t idx, const Words4& w, uint32_t val,
                                                F between)
{
    const uint8_t* base = reinterpret_cast<const uint8_t*>(lut.e);
    const uint2 lo = *reinterpret_cast<const uint2*>(base + udot4(idx, W0 | (W1 << 8), 0u));
    const uint2 hi = *reinterpret_cast<const uint2*>(base + udot4(idx, (W0 << 16) | (W1 << 24), 0u));
    between();
    const bool a0 = w.w[0] <= lo.x, a1 = w.w[1] <= lo.y, a2 = w.w[2] <= hi.x, a3 = w.w[3] <= hi.y;
    const uint32_t f0 = a0 ? val & 0xFFu : 0u, f1 = a1 ? val & 0xFF00u : 0u;
    const uint32_t f2 = a2 ? val & 0xFF0000u : 0u, f3 = a3 ? val & 0xFF000000u : 0u;
    return (f0 | f1 | f2) | f3;
}

// Spin-1: entry row (2z + 1) + nsum + z, row = ds_index(s' - s) in 0 .. 3.
struct OneLut {
    uint32_t e[52];     // thr - 1
    uint32_t live[52];  // all ones, 0 where thr is 0 (read only if a table has such)
};

// Called by all threads of the block (the first wave writes); returns whether
// the table has a zero threshold, the same in every lane.
template <int DIM>
__device__ __forceinline__ bool build_one_lut(OneLut& lut, const uint64_t* table)
{
    constexpr uint32_t n = 4 * (4 * DIM + 1);
    const uint32_t t = threadIdx.x & 63u;
    const uint64_t thr = table[t < n ? t : 0u];
    if (threadIdx.x < n) {
        lut.e[t] = (uint32_t)(thr - 1ull);
        lut.live[t] = thr == 0 ? 0u : ~0u;
    }
    return __builtin_amdgcn_ballot_w64(thr == 0) != 0ull;
}

// New s + 1 of four sites.  q: s + 1; S: nsum + z; words wa (sites 0 and 1) and
// wb: acceptance and proposal word of each site; f: 0xFF per accepted site.
// ZERO: the table may hold zero thresholds (a path of its own: a branch here
// keeps the compiler from overlapping the words of a lane).
template <int DIM, bool ZERO, class F>
__device__ __forceinline__ uint32_t one_move(uint32_t q, uint32_t S, const Words4& wa, const Words4& wb,
                                             const OneLut& lut, uint32_t& f, F between)
{
    constexpr uint32_t row = 4u * (4u * DIM + 1u);  // bytes of a table row
    // selector 2 (s + 1) + (top bit of the proposal word)
    const uint32_t t1 = __builtin_amdgcn_perm(wa.w[3], wa.w[1], 0x0C0C0703u);
    const uint32_t t2 = __builtin_amdgcn_perm(wb.w[3], wb.w[1], 0x07030C0Cu);
    const uint32_t sel = (q << 1) | (((t1 | t2) & 0x80808080u) >> 7);
    // by selector, s' + 1 and the table row: s = -1 -> 0, +1; 0 -> -1, +1; +1 -> -1, 0
    const uint32_t cand = __builtin_amdgcn_perm(0x00000100u, 0x02000201u, sel);
    const uint32_t rows = __builtin_amdgcn_perm(row << 8, (2u * row) | ((3u * row) << 8) | (row << 16) |
                                                ((2u * row) << 24), sel);
    const uint32_t idx = (S << 2) + rows;
    const uint8_t* base = reinterpret_cast<const uint8_t*>(lut.e);
    const uint8_t* live = reinterpret_cast<const uint8_t*>(lut.live);
    uint32_t t[4], on[4], b4[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const uint32_t at = (idx >> (8 * b)) & 0xFFu;
        t[b] = *reinterpret_cast<const uint32_t*>(base + at);
        on[b] = ZERO ? *reinterpret_cast<const uint32_t*>(live + at) : ~0u;
    }
    between();
#pragma unroll
    for (int b = 0; b < 4; ++b) b4[b] = (b < 2 ? wa : wb).w[(b & 1) * 2] <= t[b] ? on[b] & (0xFFu << (8 * b)) : 0u;
    f = (b4[0] | b4[1] | b4[2]) | b4[3];
    return (cand & f) | (q & ~f);
}

// s from s + 1 in every byte
__device__ __forceinline__ uint32_t spin_of(uint32_t q) { return (q + 0x7F7F7F7Fu) ^ 0x80808080u; }

}  // namespace spinlat
