// kernels_tile_ne.hip -- tile kernels of North-East lattices, J = 0 and with
// the Ising coupling (tile_device.hpp).
#include "tile_kernels.h"

namespace spinlat {

hipError_t launch_tile_ne(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                          hipStream_t s)
{
    if (a.lut_n > 2) return tilek::launch_k<tilek::KIND_NE_COUPLED, 2>(a, tg, k, dst0, dst1, s);
    return tilek::launch_k<KIND_NE, 2>(a, tg, k, dst0, dst1, s);
}

}  // namespace spinlat
