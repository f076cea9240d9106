// kernels_plane.hip -- the 3D walk along z for single lattices (plane_device.hpp).
#include "block_order.hpp"
#include "plane_device.hpp"

namespace spinlat {

namespace {

uint32_t cdiv(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

template <int KIND, int IPT>
__global__ void __launch_bounds__(tilek::kMaxBlock) k_plane(SweepArgs a, PlaneGeom pg, uint8_t* dst0, uint8_t* dst1)
{
    __shared__ planek::PlaneLds<IPT> lds;
    int32_t v[kQ];
    const uint32_t item = xcd_item(blockIdx.x, gridDim.x);
    const uint32_t tz = item / pg.nty, z0 = tz * pg.Hz;
    planek::plane_run<KIND, IPT>(a, pg, item - tz * pg.nty, z0, min(pg.Hz, pg.L - z0), dst0, dst1, a.lut, lds, v);
    block_accumulate(v[0], v[1], v[2], v[3], a.acc);
}

}  // namespace

bool plane_geom(const Geom& g, uint32_t H, uint32_t Hz, PlaneGeom& p, uint32_t max_items)
{
    p = PlaneGeom{};
    if (g.dim != 3 || !H || !Hz) return false;
    p.L = g.L;
    p.ncols = g.Lh / 4;
    p.H = H < g.L ? H : g.L;
    p.hy = p.H == g.L ? 0 : 2;
    p.RY = p.H + 2 * p.hy;
    p.Hz = Hz < g.L ? Hz : g.L;
    if (p.H + p.hy > g.L) return false;
    p.nitems = p.RY * p.ncols;
    if (p.nitems > max_items) return false;
    p.nty = cdiv(g.L, p.H);
    p.ntz = cdiv(g.L, p.Hz);
    p.magicP = (uint32_t)(((1ull << 32) + p.ncols - 1) / p.ncols);
    p.ipt = p.nitems <= 1024 ? 1 : 2;
    p.block = cdiv(cdiv(p.nitems, p.ipt), 64) * 64;
    return true;
}

// Column size by a cost model fitted to 300 timings on MI355X (6% rms): the
// launch, then per step a constant and a share per wave that the fullest SIMD
// holds.  One workgroup per CU at most: a second round of columns was never
// faster.  It puts spin-1/2 L = 200 (34 rows x 5 planes) at 10.4 us per sweep
// (measured 11.6), spin-1 L = 240 (30 x 8) at 20.0 (21.4).
bool plane_plan(const Geom& g, int kind, PlaneGeom& best)
{
    const bool one = kind == KIND_ISING_ONE;
    const double launch = one ? 2.5 : 3.26, step = one ? 0.49 : 0.34, wave = one ? 0.314 : 0.172,
                 two = one ? 1.07 : 1.13;  // two words per thread
    double best_us = 1e30;
    for (uint32_t nty = 1; nty <= 256; ++nty) {
        const uint32_t H = cdiv(g.L, nty);
        if (H < 8) break;
        const uint32_t ntz = 256 / cdiv(g.L, H);
        PlaneGeom p;
        if (!ntz || !plane_geom(g, H, cdiv(g.L, ntz), p)) continue;
        const double waves = cdiv(p.block / 64, 4) * p.ipt;
        const double us = launch + (p.Hz + 2) * (step + wave * waves * (p.ipt == 2 ? two : 1.0));
        if (us < best_us) {
            best_us = us;
            best = p;
        }
    }
    return best_us < 1e30;
}

hipError_t launch_plane(const SweepArgs& a, int kind, const PlaneGeom& pg, uint8_t* dst0, uint8_t* dst1, hipStream_t s)
{
    const dim3 grid(pg.nty * pg.ntz), block(pg.block);
    if (kind == KIND_ISING_HALF) {
        if (pg.ipt == 1) hipLaunchKernelGGL((k_plane<KIND_ISING_HALF, 1>), grid, block, 0, s, a, pg, dst0, dst1);
        else hipLaunchKernelGGL((k_plane<KIND_ISING_HALF, 2>), grid, block, 0, s, a, pg, dst0, dst1);
    } else if (kind == KIND_ISING_ONE) {
        if (pg.ipt == 1) hipLaunchKernelGGL((k_plane<KIND_ISING_ONE, 1>), grid, block, 0, s, a, pg, dst0, dst1);
        else hipLaunchKernelGGL((k_plane<KIND_ISING_ONE, 2>), grid, block, 0, s, a, pg, dst0, dst1);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace spinlat
