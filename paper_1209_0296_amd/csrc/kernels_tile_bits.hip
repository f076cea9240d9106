// kernels_tile_bits.hip -- tile launches of large North-East lattices (J = 0) on
// bit words: several sweeps of a tile per launch, as in tile_device.hpp, with 32
// same-colour sites of a row per word.
//
// What bounds it: the latency of a half-sweep (0.85 us, of which listing, reading the
// list and drawing are most), and instructions.  A site moves only if its north and
// east neighbours are occupied, and then draws only if its threshold is below 2^32:
// at c = 0.1 about 4% of the 4-site groups that share a Philox call do.  Lanes that
// hold one group each draw whenever any of a wave's 64 groups needs it, which is
// nearly always (83 instructions per group and half-sweep); here a lane holds 8 groups
// per word, the bookkeeping of which is 35 instructions, and a wave lists the groups
// that draw and shares them out, one per lane.  L = 4096, c = 0.1: 13.6 us per sweep
// before, 3.5 now; at c = 0.3, where a quarter of the groups draws, 13.6 and 6.3; where
// no move draws (c = 1/2) 7.6 and 2.2.  (Rows read and written 4 instead of 16 bytes a
// time: 4.9.)
//
// A thread owns IPT words of each colour at the same place of both colours:
// occupations and flags in registers, occupations also in LDS for the neighbours.
// Bit 4 g + b of a word is site b of 4-byte group g, the tile's words 8 groups
// each from its first column on, wrapping around the row group by group: a row
// need not be a whole number of words.  The halo in x is a word (8 groups, 32 sites
// of a colour), of which every half-sweep invalidates one site.
#include "block_order.hpp"
#include "philox.hpp"
#include "site_update.hpp"
#include "spinlat_internal.h"
#include "tile_kernels.h"

namespace spinlat {
namespace tilebits {

constexpr int kMaxBlock = 1024;
constexpr int kFlush = 8;  // sweeps whose sums LDS holds
constexpr int kObsSlots = 32;

template <int IPT>
struct BitsLds {
    uint32_t q[2][IPT * kMaxBlock];         // occupations
    uint32_t drawn[IPT * kMaxBlock];        // by word: bit 4 g + b set if the site's number is below the threshold
    uint2 place[IPT * kMaxBlock];           // by word: first group of its lattice row; its own first column
    uint16_t list[kMaxBlock / 64][IPT * 64 * 8];  // by wave: groups that draw, 32 (64 i + lane) + 4 g
    int32_t obs[kFlush][kQ][kObsSlots];
};

// Sums over the lanes up to and including each.
__device__ __forceinline__ int32_t wave_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // lane 15 of rows 0 and 2 to the next
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // lane 31 to rows 2 and 3
    return v;
}

// Bit K of the four bytes of v as bits 0 .. 3.
template <int K>
__device__ __forceinline__ uint32_t gather4(uint32_t v)
{
    return __builtin_amdgcn_udot4(v & (0x01010101u << K), 0x08040201u, 0u, false) >> K;
}

// Bits 0 .. 3 of v as bit 0 of four bytes.
__device__ __forceinline__ uint32_t scatter4(uint32_t v)
{
    return __umul24(v & 0xFu, 0x204081u) & 0x01010101u;
}

// VEC: rows of a multiple of four groups (L of 32), read and written 16 bytes at
// a time.
template <int IPT, bool VEC>
__global__ void __launch_bounds__(kMaxBlock) k_tile_bits(SweepArgs a, TileGeom tg, uint32_t nsweeps, uint8_t* dst0,
                                                         uint8_t* dst1)
{
    __shared__ BitsLds<IPT> lds;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    const uint32_t tile = xcd_item(blockIdx.x, gridDim.x);
    const uint32_t ty = tile / tg.ntx, tx = tile - ty * tg.ntx;
    const uint32_t x0 = tx * tg.W, y0 = ty * tg.H;
    const uint32_t wi = min(tg.W, tg.ncols - x0), hi = min(tg.H, tg.L - y0);
    const uint32_t PW = tg.P / 8;

    uint32_t n[2][IPT], flag[2][IPT], at[IPT], msk[IPT], col0[IPT], row0[IPT];
    int32_t depth[IPT];
    bool odd[IPT];
    int sites = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        // a wave's words are neighbours
        const uint32_t item0 = (wave * IPT + (uint32_t)i) * 64u + lane;
        const bool ok = item0 < tg.nitems;
        const uint32_t item = ok ? item0 : 0u;
        const uint32_t r = __umulhi(item, tg.magicP), w = item - r * PW;
        uint32_t gx = x0 + 8 * w + tg.ncols - tg.hx, gy = y0 + r + tg.L - tg.hy;
        gx = gx >= 2 * tg.ncols ? gx - 2 * tg.ncols : gx >= tg.ncols ? gx - tg.ncols : gx;
        gy = gy >= 2 * tg.L ? gy - 2 * tg.L : gy >= tg.L ? gy - tg.L : gy;
        at[i] = item;
        col0[i] = gx;
        row0[i] = gy * tg.ncols;
        odd[i] = (gy & 1u) != 0;
        depth[i] = ok ? (int32_t)min(r, tg.RY - 1 - r) : -1;
        // groups of the tile itself
        const int32_t left = (int32_t)wi - (int32_t)(8 * w - tg.hx);
        const bool in = ok && w > 0 && r - tg.hy < hi && left > 0;
        msk[i] = !in ? 0u : left >= 8 ? ~0u : (1u << (4 * left)) - 1u;
        sites += __builtin_popcount(msk[i]);
        uint32_t v[2][8];
        if (VEC) {
            const uint32_t x4 = gx + 4, col4 = x4 >= tg.ncols ? x4 - tg.ncols : x4;
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int g = 0; g < 8; g += 4) {
                    const uint4 u = *reinterpret_cast<const uint4*>(a.col[c] + 4ull * (row0[i] + (g ? col4 : gx)));
                    v[c][g] = u.x, v[c][g + 1] = u.y, v[c][g + 2] = u.z, v[c][g + 3] = u.w;
                }
        } else {
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const uint32_t x = gx + g, col = x >= tg.ncols ? x - tg.ncols : x;
                const uint64_t off = 4ull * (row0[i] + col);
                v[0][g] = *reinterpret_cast<const uint32_t*>(a.col[0] + off);
                v[1][g] = *reinterpret_cast<const uint32_t*>(a.col[1] + off);
            }
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n[c][i] = flag[c][i] = 0;
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                n[c][i] |= gather4<0>(v[c][g]) << (4 * g);
                flag[c][i] |= gather4<1>(v[c][g]) << (4 * g);
            }
        }
    }
    for (uint32_t e = tid; e < kFlush * kQ * kObsSlots; e += blockDim.x) (&lds.obs[0][0][0])[e] = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t slot = (wave * IPT + (uint32_t)i) * 64u + lane;
        lds.q[0][slot] = n[0][i];
        lds.q[1][slot] = n[1][i];
        lds.drawn[slot] = 0;
        lds.place[slot] = make_uint2(row0[i], col0[i]);
    }
    const PhiloxKey ks = philox_schedule(a.key0, a.key1);
    // one of the two thresholds at most is below 2^32
    const uint64_t thr_up = a.lut[0], thr_down = a.lut[1];
    const bool up_rand = thr_up < (1ull << 32), any_rand = up_rand || thr_down < (1ull << 32);
    const uint32_t thr = (uint32_t)(up_rand ? thr_up : thr_down);
    const uint32_t draw_if = any_rand ? ~0u : 0u, empty = up_rand ? ~0u : 0u;
    uint16_t* list = lds.list[wave];
    const uint32_t wave0 = wave * IPT * 64u;
    __syncthreads();

    for (uint32_t s = 0; s < nsweeps; ++s) {
        int32_t v[kQ] = {0, 0, 0, 2 * sites};
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const PhiloxSweep sw = philox_sweep((uint32_t)c, a.t + s, ks);
            const int32_t j = (int32_t)(2 * s) + c;
            const uint32_t* q = lds.q[c ^ 1];
            uint32_t allowed[IPT], rnd[IPT], pend[IPT], nb[IPT][3];
            int32_t count = 0;
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                const bool on = depth[i] > j;
                const uint32_t up = on ? at[i] - PW : at[i], down = on ? at[i] + PW : at[i];
                // the horizontal neighbours: the word itself, and that with the sites
                // moved by one, to the east where the row's colour starts the pairs
                const bool east = odd[i] == (c == 0);
                const uint32_t side = east ? at[i] + 1u : at[i] - 1u;
                const uint32_t qu = q[up], qd = q[down], qs = q[on ? side : at[i]];
                const uint32_t same = n[c ^ 1][i];
                const uint32_t moved = east ? __builtin_amdgcn_alignbit(qs, same, 1)
                                            : __builtin_amdgcn_alignbit(same, qs, 31);
                nb[i][0] = qu;
                nb[i][1] = qd;
                nb[i][2] = moved;
                allowed[i] = on ? qu & (east ? moved : same) : 0u;
                rnd[i] = allowed[i] & (n[c][i] ^ empty) & draw_if;
                const uint32_t two = rnd[i] | (rnd[i] >> 1);
                pend[i] = (two | (two >> 2)) & 0x11111111u;
                count += __builtin_popcount(pend[i]);
            }
            const int32_t upto = wave_scan(count);
            const int32_t total = __builtin_amdgcn_readlane(upto, 63);
            if (total != 0) {
                // list the wave's groups that draw
                uint32_t p = (uint32_t)(upto - count);
#pragma unroll
                for (int i = 0; i < IPT; ++i)
                    for (uint32_t left = pend[i]; left != 0u; left &= left - 1u)
                        list[p++] = (uint16_t)(32u * (64u * i + lane) + (uint32_t)__builtin_ctz(left));
                asm volatile("" ::: "memory");  // the wavefront's LDS instructions run in order
                // an entry and its word's place are read while the one before is drawn
                uint32_t x = list[min((int32_t)lane, total - 1)];
                uint2 pl = lds.place[wave0 + (x >> 5)];
                for (int32_t e = (int32_t)lane; e < total; e += 64) {
                    const uint32_t xn = list[min(e + 64, total - 1)];
                    const uint32_t cx = pl.y + ((x >> 2) & 7u);
                    const uint32_t grp = pl.x + (cx >= tg.ncols ? cx - tg.ncols : cx);
                    const Words4 wa = philox_words(philox_site(grp, 0u, ks), sw, ks);
                    uint32_t lt = 0;
#pragma unroll
                    for (int b = 3; b >= 0; --b) lt = lt + lt + (wa.w[b] < thr ? 1u : 0u);
                    atomicOr(&lds.drawn[wave0 + (x >> 5)], lt << (x & 31u));
                    x = xn;
                    pl = lds.place[wave0 + (x >> 5)];
                }
                asm volatile("" ::: "memory");
            }
#pragma unroll
            for (int i = 0; i < IPT; ++i) {
                uint32_t f = allowed[i];
                if (rnd[i] != 0u) {
                    f &= lds.drawn[at[i]] | ~rnd[i];
                    lds.drawn[at[i]] = 0;
                }
                n[c][i] ^= f;
                flag[c][i] |= f;
                if (depth[i] > j) lds.q[c][at[i]] = n[c][i];
                const uint32_t no = n[c][i] & msk[i];
                v[1] += __builtin_popcount(no);
                v[2] += __builtin_popcount(f & msk[i]);
                v[3] -= __builtin_popcount(flag[c][i] & msk[i]);
                if (c == 1)
                    v[0] += __builtin_popcount(no & nb[i][0]) + __builtin_popcount(no & nb[i][1]) +
                            __builtin_popcount(no & nb[i][2]) + __builtin_popcount(no & n[0][i]);
            }
            if (c == 1 && sites != 0) {
                int32_t(*slot)[kObsSlots] = lds.obs[s % kFlush];
#pragma unroll
                for (int k = 0; k < kQ; ++k) atomicAdd(&slot[k][tid % kObsSlots], v[k]);
            }
            __syncthreads();
        }
        const uint32_t held = s % kFlush + 1;
        if (held == kFlush || s + 1 == nsweeps) {
            // sums of the last `held` sweeps; the next additions to a slot come
            // after a barrier that every thread passes behind this
            for (uint32_t e = tid; e < held * kQ * kObsSlots; e += blockDim.x) {
                int32_t* p = &lds.obs[0][0][0] + e;
                int32_t x = *p;
                *p = 0;
#pragma unroll
                for (int off = kObsSlots / 2; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
                if (e % kObsSlots == 0 && x != 0) {
                    const uint32_t k = e / (kQ * kObsSlots), qn = (e / kObsSlots) % kQ;
                    atomicAdd(a.acc + (uint64_t)(s + 1 - held + k) * kSlotWords + (tile % kSub) * kSubStride + qn,
                              (unsigned long long)(int64_t)x);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        if (msk[i] == 0u) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            uint8_t* dst = (c ? dst1 : dst0) + 4ull * (row0[i] + col0[i]);  // the tile itself does not wrap
            uint32_t v[8];
#pragma unroll
            for (int g = 0; g < 8; ++g)
                v[g] = scatter4(n[c][i] >> (4 * g)) | scatter4(flag[c][i] >> (4 * g)) << 1;
            if (VEC) {  // groups in fours, as the row's
                *reinterpret_cast<uint4*>(dst) = make_uint4(v[0], v[1], v[2], v[3]);
                if (msk[i] >> 16) *reinterpret_cast<uint4*>(dst + 16) = make_uint4(v[4], v[5], v[6], v[7]);
            } else {
#pragma unroll
                for (int g = 0; g < 8; ++g)
                    if ((msk[i] >> (4 * g)) & 1u) *reinterpret_cast<uint32_t*>(dst + 4 * g) = v[g];
            }
        }
    }
}

template <int IPT>
hipError_t launch(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1, hipStream_t s)
{
    const dim3 grid(tg.ntx * tg.nty), block(tg.block);
    if (tg.ncols % 4 == 0)
        hipLaunchKernelGGL((k_tile_bits<IPT, true>), grid, block, 0, s, a, tg, k, dst0, dst1);
    else
        hipLaunchKernelGGL((k_tile_bits<IPT, false>), grid, block, 0, s, a, tg, k, dst0, dst1);
    return hipGetLastError();
}

}  // namespace tilebits

hipError_t launch_tile_bits(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                            hipStream_t s)
{
    if ((uint64_t)tg.block * tg.ipt < tg.nitems || tg.block > (uint32_t)tilebits::kMaxBlock || tg.P % 8 || tg.hx != 8 ||
        2 * k > 32 || tg.hy != 2 * k || tg.wrapx || tg.wrapy)
        return hipErrorInvalidValue;
    return tg.ipt == 1   ? tilebits::launch<1>(a, tg, k, dst0, dst1, s)
           : tg.ipt == 2 ? tilebits::launch<2>(a, tg, k, dst0, dst1, s)
                         : hipErrorInvalidValue;
}

}  // namespace spinlat
