// kernels_simple.hip -- initial state, layout conversion, the record of a
// lattice as it is, record folding, the overlap reduction, the direct (no LDS)
// half-sweep kernel and the resident kernel that runs many sweeps of a small
// lattice held in LDS (tables with zero thresholds, and lattices beyond a
// tile), for gfx950.
//
// Layout: two colour arrays of L^dim/2 int8 sites (see spinlat_internal.h).
// One thread owns one 4-byte word = 4 consecutive same-colour sites of one row
// (Lh % 4 == 0), which is exactly the set of sites one Philox4x32-10 call
// serves for one-word moves (spin-1/2, NE) and two calls serve for spin-1.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "philox.hpp"
#include "site_update.hpp"
#include "simple_device.hpp"
#include "spinlat_internal.h"

namespace spinlat {

using namespace simplek;

namespace {

constexpr int kBlock = 256;

// ---------------------------------------------------------------------------
// A thread of the kernels below owns the words of both colours at one place:
// words g of the two arrays hold sites x = 8 col .. 8 col + 7 of row g / ncols,
// which are bytes 8 g .. 8 g + 7 of the natural order.  So a lattice moves
// between the two layouts in 8-byte pieces, interleaved in registers: a copy of
// 2D L = 8192 takes 21.7 us (134 MB, 6.2 TB/s out of the last-level cache)
// where single bytes, two apart, took 107.

// Parity of colour 0 in a row: which of the 8 sites are its four.  L is even,
// so row = z L + y has the parity of y.
__device__ __forceinline__ bool odd_row(const Geom& g, uint32_t word)
{
    const uint32_t row = word / (g.Lh >> 2);
    return ((row + (g.dim == 3 ? row / g.L : 0u)) & 1u) != 0;
}

// 8 sites in x order from the four at even x (e) and the four at odd x (o).
__device__ __forceinline__ uint2 interleave(uint32_t e, uint32_t o)
{
    return make_uint2(__builtin_amdgcn_perm(o, e, 0x05010400u), __builtin_amdgcn_perm(o, e, 0x07030602u));
}
__device__ __forceinline__ void split(uint2 v, uint32_t& e, uint32_t& o)
{
    e = __builtin_amdgcn_perm(v.y, v.x, 0x06040200u);
    o = __builtin_amdgcn_perm(v.y, v.x, 0x07050301u);
}

// The 8 natural bytes of place g; `aligned`: the caller's buffer is 8-byte
// aligned (it need not be).
__device__ __forceinline__ uint2 load_natural(const int8_t* nat, uint64_t g, bool aligned)
{
    if (aligned) return *reinterpret_cast<const uint2*>(nat + 8 * g);
    const uint8_t* p = reinterpret_cast<const uint8_t*>(nat) + 8 * g;
    uint2 v = make_uint2(0u, 0u);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        v.x |= (uint32_t)p[b] << (8 * b);
        v.y |= (uint32_t)p[4 + b] << (8 * b);
    }
    return v;
}

__device__ __forceinline__ void natural_words(const Geom& geom, const int8_t* nat, uint64_t g, bool aligned,
                                              uint32_t& w0, uint32_t& w1)
{
    uint32_t e, o;
    split(load_natural(nat, g, aligned), e, o);
    const bool odd = odd_row(geom, (uint32_t)g);  // then colour 0 holds the odd x
    w0 = odd ? o : e;
    w1 = odd ? e : o;
}

// Word g of colour c of a random or cold start (Alg. I step 1; NE: up with
// probability c, Sec. 3.2), drawn from Philox with tag 1 at sweep 0.
template <int KIND>
__device__ __forceinline__ uint32_t start_word(uint32_t g, uint32_t c, bool random, uint64_t thr, const PhiloxKey& ks)
{
    const Words4 r = philox4x32_10(g, c, 0u, 1u, ks);
    uint32_t word = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const uint32_t u = r.w[b];
        int v;
        if (KIND == KIND_NE) v = ((uint64_t)u < thr) ? 1 : 0;
        else if (!random) v = 1;
        else if (KIND == KIND_ISING_HALF) v = (u < 0x80000000u) ? 1 : -1;
        else v = (int)(((uint64_t)u * 3u) >> 32) - 1;
        word |= ((uint32_t)(uint8_t)(int8_t)v) << (8 * b);
    }
    return word;
}

// Everything a new lattice needs before its first record, in one launch: the
// start, a cleared record ring, and the host's tables (passed by value, so that
// no copy and no staging buffer outlive the call).
template <int KIND>
__global__ void __launch_bounds__(kBlock) k_start(StartArgs s, StartBlob blob)
{
    const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < s.blob_words) s.blob_dst[threadIdx.x] = blob.w[threadIdx.x];
    for (uint64_t i = g; i < s.ring_words; i += (uint64_t)gridDim.x * kBlock) s.ring[i] = 0ull;
    if (g >= s.a.g.nh >> 2) return;
    uint32_t w0, w1;
    if (s.nat) {
        natural_words(s.a.g, s.nat, g, s.aligned != 0, w0, w1);
    } else {
        const PhiloxKey ks = philox_schedule(s.a.key0, s.a.key1);
        w0 = start_word<KIND>((uint32_t)g, 0u, s.random != 0, s.thr, ks);
        w1 = start_word<KIND>((uint32_t)g, 1u, s.random != 0, s.thr, ks);
    }
    *reinterpret_cast<uint32_t*>(s.a.col[0] + 4 * g) = w0;
    *reinterpret_cast<uint32_t*>(s.a.col[1] + 4 * g) = w1;
}

__global__ void __launch_bounds__(kBlock) k_to_natural(SweepArgs a, int8_t* nat, int aligned)
{
    const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g >= a.g.nh >> 2) return;
    const uint32_t w0 = *reinterpret_cast<const uint32_t*>(a.col[0] + 4 * g);
    const uint32_t w1 = *reinterpret_cast<const uint32_t*>(a.col[1] + 4 * g);
    const bool odd = odd_row(a.g, (uint32_t)g);
    const uint2 v = odd ? interleave(w1, w0) : interleave(w0, w1);
    if (aligned) {
        *reinterpret_cast<uint2*>(nat + 8 * g) = v;
        return;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        nat[8 * g + b] = (int8_t)(uint8_t)(v.x >> (8 * b));
        nat[8 * g + 4 + b] = (int8_t)(uint8_t)(v.y >> (8 * b));
    }
}

// Overlap sum_i v_i v_i^ref with a natural-order reference lattice (v = s for
// Ising, 2n - 1 for an NE occupation n), accumulated into one int64.
__global__ void __launch_bounds__(kBlock) k_overlap(SweepArgs a, const int8_t* ref, int aligned, int ne,
                                                    unsigned long long* out)
{
    const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    int32_t sum = 0;
    if (g < a.g.nh >> 2) {
        uint32_t r[2];
        natural_words(a.g, ref, g, aligned != 0, r[0], r[1]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const uint32_t w = *reinterpret_cast<const uint32_t*>(a.col[c] + 4 * g);
            // NE: a site counts +1 where the occupations agree, else -1
            if (ne) sum += 4 - 2 * __builtin_popcount((w ^ r[c]) & 0x01010101u);
            else sum = __builtin_amdgcn_sdot4((int)w, (int)r[c], sum, false);
        }
    }
    __shared__ int32_t part[kBlock / 64];
    sum = wave_sum(sum);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t t = 0;
        for (int w = 0; w < kBlock / 64; ++w) t += part[w];
        if (t != 0) atomicAdd(out, (unsigned long long)t);
    }
}

// Record of a lattice as it is: bond sum (over the sites of colour 1, which
// take part in every bond once), magnetisation and NE sites never flipped.
template <int KIND, int DIM>
__global__ void __launch_bounds__(kBlock) k_observe(SweepArgs a)
{
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    int32_t bond = 0, mag = 0, unfl = 0;
    if (g < (uint32_t)(a.g.nh >> 2)) {
        const uint32_t ncols = a.g.Lh >> 2, L = a.g.L;
        const uint32_t row = g / ncols, col = g - row * ncols;
        const uint32_t z = DIM == 3 ? row / L : 0u, y = row - z * L;
        const uint32_t* w0 = reinterpret_cast<const uint32_t*>(a.col[0]);
        const uint32_t own = reinterpret_cast<const uint32_t*>(a.col[1])[g];
        const uint32_t same = w0[g];
        // sideways neighbours: to the left in rows where colour 1 holds even x
        const bool right = ((y + z + 1) & 1u) != 0;
        const uint32_t adj = right ? w0[col + 1 == ncols ? g + 1 - ncols : g + 1] : w0[col == 0 ? g + ncols - 1 : g - 1];
        uint32_t nb[2 * DIM];
        nb[0] = same;
        nb[1] = right ? __builtin_amdgcn_alignbyte(adj, same, 1) : __builtin_amdgcn_alignbyte(same, adj, 3);
        nb[2] = w0[y == 0 ? g + (L - 1) * ncols : g - ncols];
        nb[3] = w0[y + 1 == L ? g - (L - 1) * ncols : g + ncols];
        if constexpr (DIM == 3) {
            const uint32_t pl = L * ncols;
            nb[4] = w0[z == 0 ? g + (L - 1) * pl : g - pl];
            nb[5] = w0[z + 1 == L ? g - (L - 1) * pl : g + pl];
        }
        constexpr uint32_t ones = 0x01010101u;
        const uint32_t s1 = KIND == KIND_NE ? own & ones : own, s0 = KIND == KIND_NE ? same & ones : same;
#pragma unroll
        for (int k = 0; k < 2 * DIM; ++k)
            bond = __builtin_amdgcn_sdot4((int)s1, (int)(KIND == KIND_NE ? nb[k] & ones : nb[k]), bond, false);
        mag = __builtin_amdgcn_sdot4((int)s0, (int)ones, __builtin_amdgcn_sdot4((int)s1, (int)ones, 0, false), false);
        if (KIND == KIND_NE)
            unfl = 8 - __builtin_popcount(own & 0x02020202u) - __builtin_popcount(same & 0x02020202u);
    }
    block_accumulate(bond, mag, 0, unfl, a.acc);
}

__global__ void __launch_bounds__(kBlock) k_clear_flags(SweepArgs a)
{
    const uint64_t ngroups = a.g.nh >> 2;
    const uint64_t gi = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (gi >= 2 * ngroups) return;
    const uint32_t c = gi >= ngroups ? 1u : 0u;
    const uint64_t g = gi - (c ? ngroups : 0);
    uint32_t* p = reinterpret_cast<uint32_t*>(a.col[c] + 4 * g);
    *p = *p & 0x01010101u;
}

__global__ void __launch_bounds__(kBlock) k_fill_u64(unsigned long long* p, uint64_t n)
{
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// Sum the kSub sub-slots of each pending record, write {t, q0..q3} and clear
// the accumulators for reuse: a row of 16 lanes per record, a sub-slot each.
__global__ void __launch_bounds__(kBlock) k_fold(unsigned long long* acc, int64_t* out, uint64_t n,
                                                 uint64_t t_first, int ising)
{
    const uint64_t i = ((uint64_t)blockIdx.x * kBlock + threadIdx.x) / kSub;
    if (i < n) fold_record(acc + i * kSlotWords, threadIdx.x % kSub, out + i * kRecordWords, t_first + i, ising != 0);
}

// Direct half-sweep: one thread per 4-site word of colour a.colour.
template <int KIND, int DIM>
__global__ void __launch_bounds__(kBlock) k_simple_half(SweepArgs a)
{
    __shared__ uint64_t lut[kMaxLut];
    for (int i = threadIdx.x; i < a.lut_n; i += kBlock) lut[i] = a.lut[i];
    __syncthreads();

    const uint64_t ngroups = a.g.nh >> 2;
    const uint64_t gi = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    int32_t q_bond = 0, q_mag = 0, q_acc = 0, q_unfl = 0;
    if (gi < ngroups) {
        const PhiloxKey ks = philox_schedule(a.key0, a.key1);
        simple_word<KIND, DIM>(a.col[a.colour], reinterpret_cast<const int8_t*>(a.col[a.colour ^ 1u]),
                               a.g, a.colour, gi, a.t, ks, lut, KIND == KIND_NE && a.lut_n > 2,
                               q_bond, q_mag, q_acc, q_unfl);
    }
    block_accumulate(q_bond, q_mag, q_acc, q_unfl, a.acc);
}

template <int KIND, int DIM>
__global__ void __launch_bounds__(kResidentBlock) k_resident(SweepArgs a, uint32_t nsweeps)
{
    extern __shared__ __align__(16) uint8_t sm[];
    __shared__ uint64_t lut[kMaxLut];
    resident_run<KIND, DIM>(a, nsweeps, sm, lut);
}

inline unsigned blocks_for(uint64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(blocks_for(n)), dim3(kBlock), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_start(const StartArgs& s, int kind, const StartBlob& blob, hipStream_t st)
{
    if (s.blob_words > kStartBlobWords || s.blob_words > (uint32_t)kBlock) return hipErrorInvalidValue;
    // enough blocks for the sites, and for the ring of a small lattice (2 KiB a
    // record: with the two blocks of 2D L = 64 a ring of 1002 took 20 us)
    const unsigned sites = blocks_for(s.a.g.nh >> 2), ring = blocks_for(std::min<uint64_t>(s.ring_words, 1u << 18));
    const dim3 grid(std::max({sites, ring, 1u})), block(kBlock);
    if (kind == KIND_ISING_HALF) hipLaunchKernelGGL(k_start<KIND_ISING_HALF>, grid, block, 0, st, s, blob);
    else if (kind == KIND_ISING_ONE) hipLaunchKernelGGL(k_start<KIND_ISING_ONE>, grid, block, 0, st, s, blob);
    else hipLaunchKernelGGL(k_start<KIND_NE>, grid, block, 0, st, s, blob);
    return hipGetLastError();
}

hipError_t launch_observe(const SweepArgs& a, int kind, hipStream_t s)
{
    const dim3 grid(blocks_for(a.g.nh >> 2)), block(kBlock);
    if (kind == KIND_NE) hipLaunchKernelGGL((k_observe<KIND_NE, 2>), grid, block, 0, s, a);
    else if (kind == KIND_ISING_HALF && a.g.dim == 2) hipLaunchKernelGGL((k_observe<KIND_ISING_HALF, 2>), grid, block, 0, s, a);
    else if (kind == KIND_ISING_HALF) hipLaunchKernelGGL((k_observe<KIND_ISING_HALF, 3>), grid, block, 0, s, a);
    else if (a.g.dim == 2) hipLaunchKernelGGL((k_observe<KIND_ISING_ONE, 2>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_observe<KIND_ISING_ONE, 3>), grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_to_natural(const SweepArgs& a, int8_t* nat, hipStream_t s)
{
    hipLaunchKernelGGL(k_to_natural, dim3(blocks_for(a.g.nh >> 2)), dim3(kBlock), 0, s, a, nat, natural_aligned(nat));
    return hipGetLastError();
}

hipError_t launch_overlap(const SweepArgs& a, const int8_t* ref, int ne, unsigned long long* out,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_overlap, dim3(blocks_for(a.g.nh >> 2)), dim3(kBlock), 0, s, a, ref, natural_aligned(ref), ne,
                       out);
    return hipGetLastError();
}

bool resident_supported(const Geom& g) { return 2 * g.nh <= (uint64_t)kResidentLds; }

hipError_t launch_resident(const SweepArgs& a, int kind, uint32_t nsweeps, hipStream_t s)
{
    const size_t lds = (size_t)(2 * a.g.nh);
    if (lds > (size_t)kResidentLds) return hipErrorInvalidValue;
    const dim3 grid(1), block(kResidentBlock);
    if (kind == KIND_NE) {
        hipLaunchKernelGGL((k_resident<KIND_NE, 2>), grid, block, lds, s, a, nsweeps);
    } else if (a.g.dim == 2) {
        if (kind == KIND_ISING_HALF)
            hipLaunchKernelGGL((k_resident<KIND_ISING_HALF, 2>), grid, block, lds, s, a, nsweeps);
        else
            hipLaunchKernelGGL((k_resident<KIND_ISING_ONE, 2>), grid, block, lds, s, a, nsweeps);
    } else {
        if (kind == KIND_ISING_HALF)
            hipLaunchKernelGGL((k_resident<KIND_ISING_HALF, 3>), grid, block, lds, s, a, nsweeps);
        else
            hipLaunchKernelGGL((k_resident<KIND_ISING_ONE, 3>), grid, block, lds, s, a, nsweeps);
    }
    return hipGetLastError();
}

hipError_t launch_clear_flags(const SweepArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_flags, dim3(blocks_for(2 * (a.g.nh >> 2))), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_fold(unsigned long long* acc, int64_t* out, uint64_t n, uint64_t t_first,
                       int ising, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fold, dim3(blocks_for(n * kSub)), dim3(kBlock), 0, s, acc, out, n, t_first,
                       ising);
    return hipGetLastError();
}

hipError_t launch_simple_half(const SweepArgs& a, int kind, hipStream_t s)
{
    const dim3 grid(blocks_for(a.g.nh >> 2));
    const dim3 block(kBlock);
    if (kind == KIND_NE) {
        hipLaunchKernelGGL((k_simple_half<KIND_NE, 2>), grid, block, 0, s, a);
    } else if (a.g.dim == 2) {
        if (kind == KIND_ISING_HALF)
            hipLaunchKernelGGL((k_simple_half<KIND_ISING_HALF, 2>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((k_simple_half<KIND_ISING_ONE, 2>), grid, block, 0, s, a);
    } else {
        if (kind == KIND_ISING_HALF)
            hipLaunchKernelGGL((k_simple_half<KIND_ISING_HALF, 3>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((k_simple_half<KIND_ISING_ONE, 3>), grid, block, 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace spinlat
