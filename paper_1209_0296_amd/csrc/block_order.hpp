// block_order.hpp -- which part of the lattice a workgroup takes (device code).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace spinlat {

// Workgroups go to the chip's 8 XCDs in turn, each with an L2 of its own.
// Consecutive items share the rows between them, so each XCD takes a
// contiguous range: block b of n (any n) is item b / 8 of range b % 8, the
// first n % 8 ranges one item longer.  (Only grids that 8 divides were mapped
// before: walks of 3D L = 176 in 252 workgroups took 11.1 us, in 216 9.5.)
__device__ __forceinline__ uint32_t xcd_item(uint32_t b, uint32_t n)
{
    const uint32_t x = b & 7u, q = n >> 3, r = n & 7u;
    return x * q + (x < r ? x : r) + (b >> 3);
}

}  // namespace spinlat
