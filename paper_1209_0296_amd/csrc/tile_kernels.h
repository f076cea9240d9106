// tile_kernels.h -- the tile kernel and its launch, instantiated for one kind
// of lattice per translation unit (kernels_tile_*.hip).
#pragma once
#include "block_order.hpp"
#include "tile_device.hpp"

namespace spinlat {

hipError_t launch_tile_half(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                            hipStream_t s);
hipError_t launch_tile_one(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                           hipStream_t s);
hipError_t launch_tile_ne(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                          hipStream_t s);

hipError_t launch_tile_bits(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                            hipStream_t s);

namespace tilek {

template <int KIND, int DIM, int IPT>
__global__ void __launch_bounds__(kMaxBlock) k_tile(SweepArgs a, TileGeom tg, uint32_t nsweeps, uint8_t* dst0,
                                                    uint8_t* dst1)
{
    __shared__ TileLds<IPT> lds;
    tile_run<KIND, DIM, IPT>(a, tg, xcd_item(blockIdx.x, gridDim.x), nsweeps, dst0, dst1, a.lut, lds);
}

template <int KIND, int DIM>
hipError_t launch_k(const SweepArgs& a, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1, hipStream_t s)
{
    const dim3 grid(tg.ntx * tg.nty * tg.ntz), block(tg.block);
    if ((uint64_t)tg.block * tg.ipt < tg.nitems || tg.block > (uint32_t)kMaxBlock) return hipErrorInvalidValue;
    if (tg.ipt == 1) hipLaunchKernelGGL((k_tile<KIND, DIM, 1>), grid, block, 0, s, a, tg, k, dst0, dst1);
    else if (tg.ipt == 2) hipLaunchKernelGGL((k_tile<KIND, DIM, 2>), grid, block, 0, s, a, tg, k, dst0, dst1);
    else if (tg.ipt == 4) hipLaunchKernelGGL((k_tile<KIND, DIM, 4>), grid, block, 0, s, a, tg, k, dst0, dst1);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tilek
}  // namespace spinlat
