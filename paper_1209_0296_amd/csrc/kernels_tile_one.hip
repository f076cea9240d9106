// kernels_tile_one.hip -- tile kernels of spin-1 lattices (tile_device.hpp).
#include "tile_kernels.h"

namespace spinlat {

hipError_t launch_tile_one(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                            hipStream_t s)
{
    if (a.g.dim == 3) return tilek::launch_k<KIND_ISING_ONE, 3>(a, tg, k, dst0, dst1, s);
    return tilek::launch_k<KIND_ISING_ONE, 2>(a, tg, k, dst0, dst1, s);
}

}  // namespace spinlat
