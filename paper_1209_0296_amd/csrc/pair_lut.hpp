// pair_lut.hpp -- Metropolis acceptance of the four sites of a word with the
// thresholds of two sites per LDS read (device code), for spin-1/2 lattices
// and the coupled North-East model.
//
// A site has at most 16 table numbers (up to 7 neighbour counts for either
// spin), so a table of all pairs is 2 KiB: one 8-byte read gives two sites'
// thresholds, and its address is one v_dot4 of the word of table numbers with
// two byte weights.  Per word that is 2 address instructions and 2 reads
// against 4 and 4 for one site at a time.  Thresholds are kept as thr - 1
// ("accept iff word <= thr - 1"), so every one must be >= 1.
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

}  // namespace spinlat
