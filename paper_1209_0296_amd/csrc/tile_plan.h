// tile_plan.h -- geometry, choice and launch of the tile schedule: several
// sweeps of LDS tiles per launch (tile_device.hpp, kernels_tile*.hip).
#pragma once
#include "spinlat_internal.h"

namespace spinlat {

// Sizes in 4-byte
// words (x) and rows (y, z) of one colour; a dimension the tile holds whole
// has no halo and wraps around.
struct TileGeom {
    uint32_t L, ncols;         // lattice side; words of a colour row
    uint32_t W, H, Z;          // a full tile
    uint32_t hx, hy, hz;       // halo on each side
    uint32_t ntx, nty, ntz;
    uint32_t P, RY, RZ;        // words per row, rows and planes held in LDS
    uint32_t wrapx, wrapy, wrapz;
    uint32_t nitems;           // words of one colour held: P RY RZ
    uint32_t magicP, magicRY;  // ceil(2^32 / P), ceil(2^32 / RY)
    uint32_t block, ipt;       // threads per workgroup, words per thread and colour
    uint32_t bits;             // words of 32 sites (kernels_tile_bits.hip): 8 columns each; nitems and
                               // magicP count those, W, hx and P still columns
};

// The tile schedule of a lattice: tile size and sweeps per launch (k = 0: none).
struct TilePlan {
    uint32_t W, H, Z, k;
    uint32_t bits = 0;  // large North-East lattices (W a multiple of 8)
};

// The whole lattice as one tile (the resident schedule; does not fit if larger
// than a workgroup holds).
TilePlan whole_plan(const Geom& g);
constexpr uint32_t kTileWhole = 4096;  // sweeps per launch of a tile that is the whole lattice

// The tile is the whole lattice: no halo, any number of sweeps per launch.
inline bool tile_whole(const TileGeom& t) { return t.wrapx && t.wrapy && t.wrapz; }

// Geometry of launches of k sweeps with the plan's tile; false if it does not fit.
constexpr uint32_t kTileItems = 4 * 1024;  // words of one colour that a workgroup holds
bool tile_geom(const Geom& g, const TilePlan& p, uint32_t k, TileGeom& tg, uint32_t max_items = kTileItems);
// Words of one colour that half-sweep j of a launch updates, over all tiles.
uint64_t tile_words(const TileGeom& t, uint32_t j);
// Fastest plan for a lattice by the launch cost model (kernels_tile.hip).  sparse:
// North-East moves that draw are few (only up-flips draw).
TilePlan tile_plan(const Geom& g, int kind, bool coupled, bool sparse);
// Sweeps a.t .. a.t + k - 1, reading a.col and writing dst (another copy, or
// the same one where a single tile holds the lattice); record s to a.acc + s
// slots.  Needs every threshold of an Ising or coupled NE table >= 1.
hipError_t launch_tile(const SweepArgs& a, int kind, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                       hipStream_t s);

}  // namespace spinlat
