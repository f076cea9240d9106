// plane_plan.h -- geometry and launch of the 3D walk along z (plane_device.hpp).
#pragma once
#include "spinlat_internal.h"

namespace spinlat {

struct PlaneGeom {
    uint32_t L, ncols;
    uint32_t H, hy, RY;   // rows of a column, its halo on each side (0: all rows), rows held
    uint32_t Hz;          // planes of a column
    uint32_t nty, ntz;
    uint32_t nitems;      // words held per plane: RY ncols
    uint32_t magicP;      // ceil(2^32 / ncols)
    uint32_t block, ipt;
};

constexpr uint32_t kPlaneItems = 2 * 1024;  // words of a plane that a workgroup holds

bool plane_geom(const Geom& g, uint32_t H, uint32_t Hz, PlaneGeom& pg, uint32_t max_items = kPlaneItems);
// Column size for a single lattice; false if the walk does not take it.
bool plane_plan(const Geom& g, int kind, PlaneGeom& pg);
// Whether half-sweeps by row groups of 4 words a lane beat the walk.  They do where
// `least_waves` or more waves (8192: what the chip holds at once) have nearly no idle
// lane: a row of the lattice is then whole groups of 4 words, and the rows that fit a
// wave take all of its 64 lanes, spin-1, whose walk keeps fewer waves in flight, 55.
// us per sweep, rows against walks:
//   single lattices (least_waves 4096): spin-1/2 64 lanes L = 256 16.4 and 17.7, 512 83.0
//   and 84.3; 63 lanes 288 21.2 and 21.3, 224 14.0 and 13.5; 60 lanes 320 27.4 and 25.6, 384
//   42.7 and 40.2; rows of no whole groups 248 18.7 and 15.8, 264 22.0 and 17.9.  Spin-1
//   64 lanes 256 22.1 and 27.0; 63 lanes 224 17.7 and 19.4, 288 29.4 and 32.5; 60 lanes 320
//   38.2 and 40.0, 384 60.9 and 68.5; 55 lanes 352 52.7 and 54.3; 52 lanes 416 83.7 and 77.9;
//   no whole groups 240 23.1 and 21.2; 60 lanes in 3687 waves, L = 192 14.1 and 14.3, in
//   2134, L = 160 12.1 and 10.0;
//   8 jobs of a batch (8192): spin-1/2 256 95.8 and 100.5, 512 804 and 894, 384 (60 lanes) 375 and
//   374; spin-1 256 136 and 164, 288 198 and 242, 320 286 and 344, 352 438 and 470, 384 537
//   and 584, 448 855 and 1018; one job in 5576 waves, L = 224 25.0 and 20.6.
inline bool rows_beat_plane(const Geom& g, int kind, uint32_t least_waves)
{
    const uint32_t ncols = g.Lh / 4, lanes = ncols / 4;
    if (g.dim != 3 || ncols % 4 != 0 || lanes == 0 || lanes > 64) return false;
    const uint32_t per = 64 / lanes;  // rows of a wave
    return lanes * per >= (kind == KIND_ISING_ONE ? 55u : 64u) && (g.rows + per - 1) / per >= least_waves;
}

// One sweep, reading a.col and writing another copy; every threshold >= 1.
hipError_t launch_plane(const SweepArgs& a, int kind, const PlaneGeom& pg, uint8_t* dst0, uint8_t* dst1, hipStream_t s);

}  // namespace spinlat
