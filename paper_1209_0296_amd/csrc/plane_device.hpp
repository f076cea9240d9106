// plane_device.hpp -- one sweep of a 3D Ising lattice per launch by a walk along
// z (gfx950).
//
// Two half-sweep launches of a 3D lattice pay two launches and read each row's
// six neighbour rows from memory; at L = 256 that is 9 us a launch, of which
// the updates are 5.  Here a workgroup holds a column of the lattice -- H rows
// of whole words plus two halo rows on each side (none where it holds all
// rows) -- and walks along z, both colours at a time: step i updates colour 0
// of plane i from the old colour-1 planes i - 1, i, i + 1 and then colour 1 of
// plane i - 1 from the new colour-0 planes i - 2, i - 1, i.  The neighbours in
// z and the word at the same place are the thread's own registers; those
// within a plane come from LDS, which holds the old colour-1 plane i and the
// new colour-0 plane i - 1 (prepared, as in tile_device.hpp), double-buffered:
// one barrier per step.  The colour-0 planes and rows next to the column are
// recomputed (bit-identical random numbers); the sweep reads one copy of the
// lattice and writes the other.
#pragma once
#include <type_traits>

#include "plane_plan.h"
#include "tile_device.hpp"

namespace spinlat {
namespace planek {

using tilek::Carry;
using tilek::TileLut;

template <int IPT, int BLOCK = tilek::kMaxBlock>
struct PlaneLds {
    uint32_t q1[2][IPT * BLOCK];  // old colour 1, plane i
    uint32_t q0[2][IPT * BLOCK];  // new colour 0, plane i - 1
    TileLut lut;
};

__device__ __forceinline__ uint32_t wrapz(int z, uint32_t L)
{
    return (uint32_t)(z < 0 ? z + (int)L : z >= (int)L ? z - (int)L : z);
}

// State of one word column: colour-1 planes i - 1, i, i + 1 as held values (own
// word of the update at i - 1 first), colour-0 planes i - 2, i - 1 prepared.
struct Column {
    uint32_t c1a, c1b, c1c, own0, q0a, q0b;
};

// Column of the rows ty H .. and the zn planes from z0.  Reads a.col, writes dst0
// and dst1; leaves each lane's share of the record in v.  Every thread of the
// block calls this (barriers inside); blockDim.x * IPT >= pg.nitems.
template <int KIND, int IPT, int BLOCK>
__device__ __forceinline__ void plane_run(const SweepArgs& a, const PlaneGeom& pg, uint32_t ty, uint32_t z0, uint32_t zn,
                                          uint8_t* dst0, uint8_t* dst1, const uint64_t* table, PlaneLds<IPT, BLOCK>& lds,
                                          int32_t (&v)[kQ])
{
    constexpr bool one = KIND == KIND_ISING_ONE;
    const uint32_t tid = threadIdx.x;
    const uint32_t y0 = ty * pg.H;
    const uint32_t hi = min(pg.H, pg.L - y0);
    const uint32_t pl = pg.L * pg.ncols;  // words of a plane

    uint32_t at[IPT], pos[IPT], up[IPT], down[IPT], sideE[IPT], sideO[IPT], selE[IPT], selO[IPT], m[IPT];
    bool act1[IPT];
    Column st[IPT];
    int words = 0;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        const uint32_t it0 = tid + (uint32_t)i * blockDim.x;
        const bool ok = it0 < pg.nitems;
        const uint32_t it = ok ? it0 : 0u;
        const uint32_t P = pg.ncols;
        const uint32_t r = P == 1 ? it : __umulhi(it, pg.magicP), col = it - r * P;
        uint32_t gy = y0 + r + pg.L - pg.hy;
        gy = gy >= 2 * pg.L ? gy - 2 * pg.L : gy >= pg.L ? gy - pg.L : gy;
        at[i] = it;
        pos[i] = gy * P + col;
        up[i] = r == 0 ? (pg.hy ? it : it + (pg.RY - 1) * P) : it - P;
        down[i] = r + 1 == pg.RY ? (pg.hy ? it : it - (pg.RY - 1) * P) : it + P;
        const uint32_t left = col == 0 ? it + P - 1 : it - 1, right = col + 1 == P ? it + 1 - P : it + 1;
        const bool odd = (gy & 1u) != 0;
        // even planes: row parity gy & 1; odd planes: the other one
        sideE[i] = odd ? right : left;
        sideO[i] = odd ? left : right;
        selE[i] = odd ? 0x04030201u : 0x02010007u;
        selO[i] = odd ? 0x02010007u : 0x04030201u;
        const bool in = ok && r - pg.hy < hi;
        act1[i] = in;
        m[i] = in ? ~0u : 0u;
        words += in ? 1 : 0;
    }
    const uint8_t* S0 = a.col[0];
    const uint8_t* S1 = a.col[1];
    auto ld = [&](const uint8_t* base, int z, int i) {
        return *reinterpret_cast<const uint32_t*>(base + 4ull * ((uint64_t)wrapz(z, pg.L) * pl + pos[i]));
    };
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        st[i].c1a = ld(S1, (int)z0 - 2, i);
        st[i].c1b = ld(S1, (int)z0 - 1, i);
        st[i].c1c = ld(S1, (int)z0, i);
        st[i].own0 = ld(S0, (int)z0 - 1, i);
        st[i].q0a = st[i].q0b = 0u;
    }
    tilek::build_lut<KIND, 3>(lds.lut, table);
    const PhiloxKey ks = philox_schedule(a.key0, a.key1);
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
        st[i].c1a = tilek::hold<KIND>(st[i].c1a);
        st[i].c1b = tilek::hold<KIND>(st[i].c1b);
        st[i].c1c = tilek::hold<KIND>(st[i].c1c);
        st[i].own0 = tilek::hold<KIND>(st[i].own0);
    }
    Carry o = {0, 0, 0, 0, 0};
    const auto prp = [](uint32_t held) { return one ? held : tilek::prep<KIND>(held); };
    const auto step = [&](int i, auto odd_plane) {
        constexpr bool ODD = decltype(odd_plane)::value;
        const uint32_t b = (uint32_t)i & 1u;
        const bool do1 = i > (int)z0, mine = i >= (int)z0 && i < (int)(z0 + zn);
        uint32_t c1n[IPT], own0n[IPT];
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            lds.q1[b][at[j]] = prp(st[j].c1b);
            lds.q0[b][at[j]] = st[j].q0b;
            c1n[j] = ld(S1, i + 2, j);
            own0n[j] = ld(S0, i + 1, j);
        }
        lds_barrier();
        const uint32_t z = wrapz(i, pg.L), zm = wrapz(i - 1, pg.L);
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t s = ODD ? sideO[j] : sideE[j], sl = ODD ? selO[j] : selE[j];
            const uint32_t* q1 = lds.q1[b];
            const uint32_t* q0 = lds.q0[b];
            uint32_t q0n;
            {
                const uint32_t qu = q1[up[j]], qd = q1[down[j]], qs = q1[s];
                const uint32_t g = z * pl + pos[j];
                const Words4 wa = philox4x32_10(one ? 2 * g : g, 0u, a.t, 0u, ks);
                const Words4 wb = one ? philox4x32_10(2 * g + 1, 0u, a.t, 0u, ks) : wa;
                const uint32_t same = prp(st[j].c1b);
                const uint32_t S = same + __builtin_amdgcn_perm(qs, same, sl) + qu + qd + prp(st[j].c1a) + prp(st[j].c1c);
                const uint32_t nw = tilek::update<KIND, 3>(st[j].own0, S, 0u, 0u, 0, wa, wb, PhiloxSite{}, PhiloxSweep{},
                                                           ks, lds.lut, 0u, false, false, mine ? m[j] : 0u, o, [] {});
                q0n = prp(nw);
                if (mine && act1[j]) *reinterpret_cast<uint32_t*>(dst0 + 4ull * g) = tilek::unhold<KIND>(nw);
            }
            if (do1 && act1[j]) {
                const uint32_t qu = q0[up[j]], qd = q0[down[j]], qs = q0[s];
                const uint32_t g = zm * pl + pos[j];
                const Words4 wa = philox4x32_10(one ? 2 * g : g, 1u, a.t, 0u, ks);
                const Words4 wb = one ? philox4x32_10(2 * g + 1, 1u, a.t, 0u, ks) : wa;
                const uint32_t same = st[j].q0b;
                const uint32_t S = same + __builtin_amdgcn_perm(qs, same, sl) + qu + qd + st[j].q0a + q0n;
                const uint32_t nw = tilek::update<KIND, 3>(st[j].c1a, S, 0u, 0u, 1, wa, wb, PhiloxSite{}, PhiloxSweep{},
                                                           ks, lds.lut, 0u, false, false, ~0u, o, [] {});
                *reinterpret_cast<uint32_t*>(dst1 + 4ull * g) = tilek::unhold<KIND>(nw);
            }
            st[j].q0a = st[j].q0b;
            st[j].q0b = q0n;
            st[j].c1a = st[j].c1b;
            st[j].c1b = st[j].c1c;
            st[j].c1c = tilek::hold<KIND>(c1n[j]);
            st[j].own0 = tilek::hold<KIND>(own0n[j]);
        }
    };
    int i = (int)z0 - 1;
    const int end = (int)(z0 + zn);
    if (i & 1) step(i++, std::true_type{});
    for (; i + 1 <= end; i += 2) {
        step(i, std::false_type{});
        step(i + 1, std::true_type{});
    }
    if (i <= end) step(i, std::false_type{});
    tilek::finish<KIND, 3>(o, words * (int)zn, v);
}

}  // namespace planek
}  // namespace spinlat
