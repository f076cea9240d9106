// tile_device.hpp -- several sweeps of a tile of the lattice held in LDS (gfx950).
//
// What bounds small and middle lattices is not work but launches: a kernel
// that sweeps 2D L = 512 once takes 4.2 us, of which the attempts would need
// 0.1.  Here a workgroup loads a tile together with a halo, runs k sweeps on it
// between barriers and writes the tile's own sites to the lattice's other
// copy, so a launch pays for k sweeps.  Half-sweep j (0 .. 2k - 1) computes the
// sites that are at least j + 1 rows (planes) inside the loaded region, which
// after 2k half-sweeps leaves the tile itself; the random numbers depend on
// (seed, sweep, site) only, so a site that several tiles compute gets the same
// value in each.  A dimension that the tile holds whole has no halo: its
// neighbours wrap around inside LDS.  A lattice that is one tile needs no halo
// at all and runs any number of sweeps per launch (the resident schedule).
//
// A thread owns IPT 4-byte words (4 same-colour sites) of each colour, at the
// same place of both colours, for the whole launch.  Its words stay in
// registers; LDS holds what the neighbours read, in "prepared" form:
//   spin-1/2  bit 1 of each byte (2 per -1 spin), so that a sum of neighbours
//             is 2 x (number of -1 neighbours) per byte;
//   spin-1    s + 1;
//   NE        n.
// The word of the other colour at the same place is a neighbour of every site
// and is the thread's own; the others are three (3D: five) LDS reads, and the
// fourth, sideways, neighbour of each site comes from a byte permute of the
// word itself and the adjacent one.
//
// Acceptance: spin-1/2 and coupled NE look two sites' thresholds up at once
// (accept.hpp), spin-1 one site's.  All thresholds must be >= 1 ("word <=
// thr - 1"); other tables run elsewhere.
//
// Records: a lane adds its sums of a sweep to one of 32 LDS slots (no lane
// conflicts but between the two halves of a wave); every kFlush sweeps, and
// at the end, the slots are summed and added to the sweeps' records.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "accept.hpp"
#include "philox.hpp"
#include "site_update.hpp"
#include "spinlat_internal.h"
#include "tile_plan.h"

namespace spinlat {
namespace tilek {

constexpr int KIND_NE_COUPLED = 3;  // as in row_device.hpp
constexpr int kMaxBlock = 1024;
constexpr int kFlush = 8;           // sweeps whose sums LDS holds
constexpr int kObsSlots = 32;

union TileLut {
    PairLut pair;
    OneLut one;
};

struct Carry {
    int32_t acc, mag0, mag1, dd, unfl;
};

template <int KIND, int DIM>
__device__ __forceinline__ void build_lut(TileLut& lut, const uint64_t* table)
{
    if constexpr (KIND == KIND_ISING_ONE) {
        (void)build_one_lut<DIM>(lut.one, table);
    } else if constexpr (KIND == KIND_ISING_HALF || KIND == KIND_NE_COUPLED) {
        build_pair_lut<KIND == KIND_NE_COUPLED, DIM>(lut.pair, table);
    }
}

// Keeps the loads issued before it in front of the rounds that c goes through
// after it: the compiler orders them by the memory clobber and by c.
__device__ __forceinline__ void loads_first(Words4& c)
{
    asm volatile("" : "+v"(c.w[0]), "+v"(c.w[1]), "+v"(c.w[2]), "+v"(c.w[3])::"memory");
}

// Prepared form of a word (see above).
template <int KIND>
__device__ __forceinline__ uint32_t prep(uint32_t w)
{
    if constexpr (KIND == KIND_ISING_HALF) return w & 0x02020202u;
    else if constexpr (KIND == KIND_ISING_ONE) return (w ^ 0x80808080u) + 0x80808081u;  // s + 1, no carries
    else return w & 0x01010101u;
}

// What a register holds of an own word: the word itself, or s + 1 for spin-1.
template <int KIND>
__device__ __forceinline__ uint32_t hold(uint32_t w)
{
    return KIND == KIND_ISING_ONE ? prep<KIND>(w) : w;
}
template <int KIND>
__device__ __forceinline__ uint32_t unhold(uint32_t w)
{
    return KIND == KIND_ISING_ONE ? spin_of(w) : w;
}

// New held value of a word.  own: held; same, side, S: prepared other-colour
// words (S the sum of all neighbours); north, east: NE.  m: all ones for a
// counted word, else 0.
template <int KIND, int DIM, class F>
__device__ __forceinline__ uint32_t update(uint32_t own, uint32_t S, uint32_t north, uint32_t east, int colour,
                                           Words4 wa, const Words4& wb, const PhiloxSite& site, const PhiloxSweep& sw,
                                           const PhiloxKey& ks, const TileLut& lut, uint32_t thr, bool up_rand,
                                           bool any_rand, uint32_t m, Carry& o, F between)
{
    constexpr uint32_t ones = 0x01010101u;
    if constexpr (KIND == KIND_ISING_HALF) {
        const uint32_t idx = S | (own & 0x10101010u);  // 2 nd + 16 (s == -1)
        const uint32_t out = own ^ pair_accept<4, 68>(lut.pair, idx, wa, 0xFEFEFEFEu, between);
        const uint32_t om = out & m;
        o.acc = sdot4(own, om, o.acc);  // 4 - 2 x (flipped sites) per word
        if (colour == 0) {
            o.mag0 = sdot4(om, ones, o.mag0);
        } else {
            o.mag1 = sdot4(om, ones, o.mag1);
            o.dd = sdot4(om, S, o.dd);  // sum s' 2 nd
        }
        return out;
    } else if constexpr (KIND == KIND_ISING_ONE) {
        uint32_t f4;
        const uint32_t out = one_move<DIM, false>(own, S, wa, wb, lut.one, f4, between);
        const uint32_t om = out & m;
        o.acc += __builtin_popcount(f4 & m);  // 8 per accepted site
        if (colour == 0) {
            o.mag0 = sdot4(om, ones, o.mag0);  // sum s + 1
        } else {
            o.mag1 = sdot4(om, ones, o.mag1);
            o.dd = sdot4(om, S, o.dd);
            o.unfl = sdot4(S & m, ones, o.unfl);  // sum (nsum + z)
        }
        return out;
    } else {
        const uint32_t n = own & ones;
        const uint32_t allowed = north & east;
        uint32_t f = allowed;
        if constexpr (KIND == KIND_NE_COUPLED) {
            if (__builtin_amdgcn_ballot_w64(allowed != 0u) != 0ull) {
                wa = philox_words(site, sw, ks);
                f &= pair_accept<8, 136>(lut.pair, (n << 3) | S, wa, ones, [] {});
            }
        } else {
            // one of the two thresholds at most is below 2^32
            const uint32_t rnd = any_rand ? allowed & (up_rand ? ~n : n) : 0u;
            if (__builtin_amdgcn_ballot_w64(rnd != 0u) != 0ull) {
                wa = philox_words(site, sw, ks);
                uint32_t lt = 0;
#pragma unroll
                for (int b = 0; b < 4; ++b) lt |= wa.w[b] < thr ? 1u << (8 * b) : 0u;
                f &= lt | ~rnd;
            }
        }
        const uint32_t out = (own ^ f) | (f << 1);
        const uint32_t om = out & m;
        const uint32_t no = om & ones;
        o.acc += __builtin_popcount(f & m);
        if (colour == 0) {
            o.mag0 += __builtin_popcount(no);
        } else {
            o.mag1 += __builtin_popcount(no);
            o.dd = sdot4(no, S, o.dd);
        }
        o.unfl += __builtin_popcount(om & 0x02020202u);
        return out;
    }
}

// A lane's sums of one sweep in record units; words: the counted words of one
// colour that the lane owns.
template <int KIND, int DIM>
__device__ __forceinline__ void finish(const Carry& o, int words, int32_t (&v)[kQ])
{
    constexpr int z = 2 * DIM;
    if constexpr (KIND == KIND_ISING_HALF) {
        v[0] = z * o.mag1 - o.dd;
        v[1] = o.mag0 + o.mag1;
        v[2] = (8 * words - o.acc) >> 1;
        v[3] = 0;
    } else if constexpr (KIND == KIND_ISING_ONE) {
        // sum (s+1)(nsum + z) - sum (nsum + z) - z sum s
        v[0] = o.dd - o.unfl - z * (o.mag1 - 4 * words);
        v[1] = o.mag0 + o.mag1 - 8 * words;
        v[2] = o.acc >> 3;
        v[3] = 0;
    } else {
        v[0] = o.dd;
        v[1] = o.mag0 + o.mag1;
        v[2] = o.acc;
        v[3] = 8 * words - o.unfl;
    }
}

template <int IPT, int BLOCK = kMaxBlock>
struct TileLds {
    uint32_t q[2][IPT * BLOCK];
    TileLut lut;
    int32_t obs[kFlush][kQ][kObsSlots];
};

// Sweeps a.t .. a.t + nsweeps - 1 of tile `tile`: reads a.col, writes dst0 and
// dst1, adds the record of sweep s to a.acc + s slots.  Every thread of the
// block calls this (barriers inside); blockDim.x * IPT >= tg.nitems.
template <int KIND, int DIM, int IPT, int BLOCK>
__device__ __forceinline__ void tile_run(const SweepArgs& a, const TileGeom& tg, uint32_t tile, uint32_t nsweeps,
                                         uint8_t* dst0, uint8_t* dst1, const uint64_t* table, TileLds<IPT, BLOCK>& lds)
{
    const uint32_t tid = threadIdx.x;
    // the tile's place: x fastest
    const uint32_t ty = tile / tg.ntx, tx = tile - ty * tg.ntx;
    const uint32_t tz = DIM == 3 ? ty / tg.nty : 0u;
    const uint32_t x0 = tx * tg.W, y0 = (ty - (DIM == 3 ? tz * tg.nty : 0u)) * tg.H, z0 = DIM == 3 ? tz * tg.Z : 0u;
    const uint32_t wi = min(tg.W, tg.ncols - x0), hi = min(tg.H, tg.L - y0), zi = DIM == 3 ? min(tg.Z, tg.L - z0) : 1u;

    uint32_t own[2][IPT], grp[IPT], at[IPT], up[IPT], down[IPT], side[2][IPT], sel[2][IPT], msk[IPT];
    uint32_t zup[DIM == 3 ? IPT : 1], zdown[DIM == 3 ? IPT : 1];
    int32_t depth[IPT];
    bool east1[IPT];  // NE: the east neighbour of colour 0 is the side word
    int words = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t item0 = tid + (uint32_t)i * blockDim.x;
        const bool ok = item0 < tg.nitems;
        const uint32_t item = ok ? item0 : 0u;
        const uint32_t rr = tg.P == 1 ? item : __umulhi(item, tg.magicP), col = item - rr * tg.P;
        const uint32_t zz = DIM == 3 ? __umulhi(rr, tg.magicRY) : 0u, r = rr - zz * tg.RY;
        // lattice coordinates (halos wrap; a halo is at most one lattice deep)
        uint32_t gx = x0 + col + tg.ncols - tg.hx, gy = y0 + r + tg.L - tg.hy, gz = z0 + zz + tg.L - tg.hz;
        gx = gx >= 2 * tg.ncols ? gx - 2 * tg.ncols : gx >= tg.ncols ? gx - tg.ncols : gx;
        gy = gy >= 2 * tg.L ? gy - 2 * tg.L : gy >= tg.L ? gy - tg.L : gy;
        gz = DIM == 3 ? (gz >= 2 * tg.L ? gz - 2 * tg.L : gz >= tg.L ? gz - tg.L : gz) : 0u;
        const uint32_t g = (gz * tg.L + gy) * tg.ncols + gx;
        const bool odd = ((gy + gz) & 1u) != 0;  // row parity of colour 0
        grp[i] = g;
        own[0][i] = hold<KIND>(*reinterpret_cast<const uint32_t*>(a.col[0] + 4ull * g));
        own[1][i] = hold<KIND>(*reinterpret_cast<const uint32_t*>(a.col[1] + 4ull * g));
        int32_t d = 0x7FFFFFFF;
        if (!tg.wrapy) d = min(d, (int32_t)min(r, tg.RY - 1 - r));
        if (DIM == 3 && !tg.wrapz) d = min(d, (int32_t)min(zz, tg.RZ - 1 - zz));
        depth[i] = ok ? d : -1;
        const bool in = ok && col - tg.hx < wi && r - tg.hy < hi && (DIM == 2 || zz - tg.hz < zi);
        msk[i] = in ? ~0u : 0u;
        words += in ? 1 : 0;
        const uint32_t left = col == 0 ? (tg.wrapx ? item + tg.P - 1 : item) : item - 1;
        const uint32_t right = col + 1 == tg.P ? (tg.wrapx ? item + 1 - tg.P : item) : item + 1;
        at[i] = item;
        side[0][i] = odd ? right : left;
        side[1][i] = odd ? left : right;
        // bytes of (adjacent word : word): the left neighbours are the word
        // shifted up by a byte, the right ones shifted down
        sel[0][i] = odd ? 0x04030201u : 0x02010007u;
        sel[1][i] = odd ? 0x02010007u : 0x04030201u;
        east1[i] = odd;
        up[i] = r == 0 ? (tg.wrapy ? item + (tg.RY - 1) * tg.P : item) : item - tg.P;
        down[i] = r + 1 == tg.RY ? (tg.wrapy ? item - (tg.RY - 1) * tg.P : item) : item + tg.P;
        if constexpr (DIM == 3) {
            const uint32_t pl = tg.RY * tg.P;
            zup[i] = zz == 0 ? (tg.wrapz ? item + (tg.RZ - 1) * pl : item) : item - pl;
            zdown[i] = zz + 1 == tg.RZ ? (tg.wrapz ? item - (tg.RZ - 1) * pl : item) : item + pl;
        }
    }
    build_lut<KIND, DIM>(lds.lut, table);
    for (uint32_t e = tid; e < kFlush * kQ * kObsSlots; e += blockDim.x) (&lds.obs[0][0][0])[e] = 0;
    const PhiloxKey ks = philox_schedule(a.key0, a.key1);
    constexpr int kCalls = KIND == KIND_ISING_ONE ? 2 : 1;
    PhiloxSite site[IPT][kCalls];
#pragma unroll
    for (int i = 0; i < IPT; ++i)
#pragma unroll
        for (int k = 0; k < kCalls; ++k) site[i][k] = philox_site(kCalls * grp[i] + k, 0u, ks);
#pragma unroll
    for (int i = 0; i < IPT; ++i)
        if (depth[i] >= 0) {
            lds.q[0][at[i]] = KIND == KIND_ISING_ONE ? own[0][i] : prep<KIND>(own[0][i]);
            lds.q[1][at[i]] = KIND == KIND_ISING_ONE ? own[1][i] : prep<KIND>(own[1][i]);
        }
    // NE, J = 0: the one threshold below 2^32
    uint64_t thr_up = 0, thr_down = 0;
    if constexpr (KIND == KIND_NE) thr_up = table[0], thr_down = table[1];
    const bool up_rand = thr_up < (1ull << 32), any_rand = up_rand || thr_down < (1ull << 32);
    const uint32_t thr = (uint32_t)(up_rand ? thr_up : thr_down);
    // the loads end here: a wait for them inside the loop would also wait for
    // the records' atomics
#pragma unroll
    for (int i = 0; i < IPT; ++i) asm volatile("" : "+v"(own[0][i]), "+v"(own[1][i]));
    __syncthreads();

    // One word per thread is one or two waves per SIMD, where latencies count:
    // a half-sweep then draws the next one's numbers between its own LDS reads
    constexpr bool kAhead = IPT == 1 && (KIND == KIND_ISING_HALF || KIND == KIND_ISING_ONE);
    Words4 nxt[kCalls];
    if constexpr (kAhead) {
        const PhiloxSweep sw = philox_sweep(0u, a.t, ks);
#pragma unroll
        for (int k = 0; k < kCalls; ++k) nxt[k] = philox_words(site[0][k], sw, ks);
    }
    for (uint32_t s = 0; s < nsweeps; ++s) {
        Carry o = {0, 0, 0, 0, 0};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const PhiloxSweep sw = kAhead ? philox_sweep((uint32_t)(c ^ 1), a.t + s + c, ks)
                                          : philox_sweep((uint32_t)c, a.t + s, ks);
            const int32_t j = (int32_t)(2 * s) + c;
            const uint32_t* q = lds.q[c ^ 1];
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                if (depth[i] > j) {
                    const uint32_t qu = q[up[i]], qd = q[down[i]], qs = q[side[c][i]];
                    uint32_t qz = 0;
                    if constexpr (DIM == 3) qz = q[zup[i]] + q[zdown[i]];
                    // Ising: every word's numbers are drawn, while reads are in flight
                    Words4 wa = {}, wb = {};
                    if constexpr (kAhead) {
                        // half of the next rounds here, half behind the table reads
                        wa = nxt[0];
                        if constexpr (kCalls == 2) wb = nxt[kCalls - 1];
#pragma unroll
                        for (int k = 0; k < kCalls; ++k) {
                            nxt[k] = philox_start(site[0][k], sw);
                            loads_first(nxt[k]);
                            philox_rounds<2, 6>(nxt[k], sw, ks);
                        }
                    } else if constexpr (KIND == KIND_ISING_HALF || KIND == KIND_ISING_ONE) {
                        wa = philox_start(site[i][0], sw);
                        if constexpr (kCalls == 2) wb = philox_start(site[i][1], sw);
                        loads_first(wa);
                        philox_rounds<2, 10>(wa, sw, ks);
                        if constexpr (kCalls == 2) philox_rounds<2, 10>(wb, sw, ks);
                    }
                    const uint32_t same = KIND == KIND_ISING_ONE ? own[c ^ 1][i] : prep<KIND>(own[c ^ 1][i]);
                    const uint32_t sd = __builtin_amdgcn_perm(qs, same, sel[c][i]);
                    const uint32_t S = same + sd + qu + qd + qz;
                    const bool side_east = c == 0 ? east1[i] : !east1[i];
                    const uint32_t nw = update<KIND, DIM>(own[c][i], S, qu, side_east ? sd : same, c, wa, wb,
                                                          site[i][0], sw, ks, lds.lut, thr, up_rand, any_rand, msk[i],
                                                          o, [&] {
                                                              if constexpr (kAhead)
#pragma unroll
                                                                  for (int k = 0; k < kCalls; ++k) {
                                                                      loads_first(nxt[k]);
                                                                      philox_rounds<6, 10>(nxt[k], sw, ks);
                                                                  }
                                                          });
                    own[c][i] = nw;
                    lds.q[c][at[i]] = KIND == KIND_ISING_ONE ? nw : prep<KIND>(nw);
                }
            }
            if (c == 1) {
                int32_t v[kQ];
                finish<KIND, DIM>(o, words, v);
                if (words) {
                    int32_t(*slot)[kObsSlots] = lds.obs[s % kFlush];
                    atomicAdd(&slot[0][tid % kObsSlots], v[0]);
                    atomicAdd(&slot[1][tid % kObsSlots], v[1]);
                    atomicAdd(&slot[2][tid % kObsSlots], v[2]);
                    if constexpr (KIND != KIND_ISING_HALF && KIND != KIND_ISING_ONE)
                        atomicAdd(&slot[3][tid % kObsSlots], v[3]);
                }
            }
            __syncthreads();
        }
        const uint32_t held = s % kFlush + 1;
        if (held == kFlush || s + 1 == nsweeps) {
            // sums of the last `held` sweeps; the next additions to a slot come
            // after a barrier that every thread passes behind this
            for (uint32_t e = tid; e < held * kQ * kObsSlots; e += blockDim.x) {
                int32_t* p = &lds.obs[0][0][0] + e;
                int32_t v = *p;
                *p = 0;
#pragma unroll
                for (int off = kObsSlots / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
                if (e % kObsSlots == 0 && v != 0) {
                    const uint32_t k = e / (kQ * kObsSlots), qn = (e / kObsSlots) % kQ;
                    atomicAdd(a.acc + (uint64_t)(s + 1 - held + k) * kSlotWords + (tile % kSub) * kSubStride + qn,
                              (unsigned long long)(int64_t)v);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i)
        if (msk[i]) {
            *reinterpret_cast<uint32_t*>(dst0 + 4ull * grp[i]) = unhold<KIND>(own[0][i]);
            *reinterpret_cast<uint32_t*>(dst1 + 4ull * grp[i]) = unhold<KIND>(own[1][i]);
        }
}

}  // namespace tilek
}  // namespace spinlat
