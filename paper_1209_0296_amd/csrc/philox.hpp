// philox.hpp -- Philox4x32-10 for gfx950 device code.
//
// Salmon, Moraes, Dror & Shaw, "Parallel random numbers: as easy as 1, 2, 3"
// (SC'11): ten rounds of a keyed bijection on four 32-bit words.  A round
// forms the full 64-bit products of counter words 0 and 2 with two fixed odd
// multipliers, xors each high half with the opposite word pair and a round key
// word, and reorders the four results; the two key words advance by the two
// Weyl increments between rounds.  The key is uniform across a launch, so the
// ten round keys are computed once by the caller (scalar registers) and the
// lanes spend only the two 32x32->64 products and two three-way xors per round.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spinlat {

struct PhiloxKey {
    uint32_t k0[10];
    uint32_t k1[10];
};

__host__ __device__ inline PhiloxKey philox_schedule(uint32_t key0, uint32_t key1)
{
    PhiloxKey ks;
    for (int r = 0; r < 10; ++r) {
        ks.k0[r] = key0 + (uint32_t)r * 0x9E3779B9u;
        ks.k1[r] = key1 + (uint32_t)r * 0xBB67AE85u;
    }
    return ks;
}

struct Words4 {
    uint32_t w[4];
};

// a ^ b ^ c in one VALU instruction (gfx950 three-input bitwise op, truth
// table 0x96); the round key operand is wave-uniform and stays in a scalar
// register.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Counter (c0, c1, c2, c3) -> four uniform 32-bit words.  Rounds 0 and 1 are
// left to the compiler: when counter words 1-3 are uniform across the wave
// (colour, sweep, tag) it evaluates their products on the scalar unit.  From
// round 2 on every word varies per lane and each round is two 32x32->64
// multiply-adds and two three-way xors.
__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                uint32_t c3, const PhiloxKey& ks)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        uint32_t n0, n2;
        if (r < 2) {
            n0 = (uint32_t)(p1 >> 32) ^ c1 ^ ks.k0[r];
            n2 = (uint32_t)(p0 >> 32) ^ c3 ^ ks.k1[r];
        } else {
            n0 = xor3((uint32_t)(p1 >> 32), c1, ks.k0[r]);
            n2 = xor3((uint32_t)(p0 >> 32), c3, ks.k1[r]);
        }
        c1 = (uint32_t)p1;
        c3 = (uint32_t)p0;
        c0 = n0;
        c2 = n2;
    }
    Words4 out;
    out.w[0] = c0;
    out.w[1] = c1;
    out.w[2] = c2;
    out.w[3] = c3;
    return out;
}

// The same words, split by what each part depends on, for kernels that draw at
// the same sites sweep after sweep.  Round 0's product of counter word 0 and
// the product that round 1 forms from it depend on the site alone (and the
// key); the other product of each of the two rounds on the colour and the
// sweep alone, so it is wave-uniform.  What is left of rounds 0 and 1 for a
// call are two xors.
struct PhiloxSite {
    uint32_t a, b, c;
};
struct PhiloxSweep {
    uint32_t a, b, c;
};

__device__ __forceinline__ PhiloxSite philox_site(uint32_t c0, uint32_t c3, const PhiloxKey& ks)
{
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint32_t n2 = (uint32_t)(p0 >> 32) ^ c3 ^ ks.k1[0];
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)n2;
    PhiloxSite s;
    s.a = (uint32_t)(p1 >> 32) ^ ks.k0[1];
    s.b = (uint32_t)p0 ^ ks.k1[1];
    s.c = (uint32_t)p1;
    return s;
}

__device__ __forceinline__ PhiloxSweep philox_sweep(uint32_t c1, uint32_t c2, const PhiloxKey& ks)
{
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t n0 = (uint32_t)(p1 >> 32) ^ c1 ^ ks.k0[0];
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)n0;
    PhiloxSweep s;
    s.a = (uint32_t)p1;
    s.b = (uint32_t)(p0 >> 32);
    s.c = (uint32_t)p0 ^ ks.k1[2];
    return s;
}

// Rounds FROM .. TO - 1 (2 <= FROM) of the state c = counter words 0 .. 3; the
// state before round 2 comes from philox_start.
template <int FROM, int TO>
__device__ __forceinline__ void philox_rounds(Words4& c, const PhiloxSweep& sw, const PhiloxKey& ks)
{
#pragma unroll
    for (int r = FROM; r < TO; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c.w[0];
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c.w[2];
        c.w[0] = xor3((uint32_t)(p1 >> 32), c.w[1], ks.k0[r]);
        // sw.c holds counter word 3 with round 2's key word
        c.w[2] = r == 2 ? (uint32_t)(p0 >> 32) ^ sw.c : xor3((uint32_t)(p0 >> 32), c.w[3], ks.k1[r]);
        c.w[1] = (uint32_t)p1;
        c.w[3] = (uint32_t)p0;
    }
}

__device__ __forceinline__ Words4 philox_start(const PhiloxSite& st, const PhiloxSweep& sw)
{
    Words4 c;
    c.w[0] = st.a ^ sw.a;
    c.w[1] = st.c;
    c.w[2] = st.b ^ sw.b;
    c.w[3] = 0;
    return c;
}

// philox4x32_10(c0, c1, c2, c3) of the parts philox_site(c0, c3) and
// philox_sweep(c1, c2).
__device__ __forceinline__ Words4 philox_words(const PhiloxSite& st, const PhiloxSweep& sw, const PhiloxKey& ks)
{
    Words4 c = philox_start(st, sw);
    philox_rounds<2, 10>(c, sw, ks);
    return c;
}

}  // namespace spinlat
