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
// One sweep, reading a.col and writing another copy; every threshold >= 1.
hipError_t launch_plane(const SweepArgs& a, int kind, const PlaneGeom& pg, uint8_t* dst0, uint8_t* dst1, hipStream_t s);

}  // namespace spinlat
