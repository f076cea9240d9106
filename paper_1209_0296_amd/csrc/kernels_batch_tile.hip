// kernels_batch_tile.hip -- batched jobs on tiles (several sweeps per launch),
// by walks along z (both colours of a 3D sweep per launch) and whole in one
// tile (a call's sweeps per launch).
//
// At the load of a served stream the per-sweep families spent most of a launch
// on latency: a workgroup's chain of reads (work list, counters, job entry,
// geometry, table, lattice) before four words per lane of work, for two
// launches per sweep.  Here a launch does four sweeps of every 2D job, or a
// whole sweep of every 3D job with a workgroup walking many planes.
#include "batch_internal.h"
#include "plane_device.hpp"
#include "tile_device.hpp"

namespace spinlat {

using tilek::KIND_NE_COUPLED;

namespace {

// Tiles of at most 1536 words of one colour: two workgroups of 12 waves fit a
// CU at the registers that the spin-1 kernel needs.
constexpr int kTileBlock = 768, kTileIpt = 2;
// Whole lattices of at most 2048 words of one colour (2D L = 128, 3D L = 24).
constexpr int kWholeBlock = 512, kWholeIpt = 4;

__device__ __forceinline__ SweepArgs job_args(const BatchJob& J, uint32_t copy, uint32_t t, uint32_t slot)
{
    SweepArgs a{};
    a.col[0] = copy ? J.col[1][0] : J.col[0][0];
    a.col[1] = copy ? J.col[1][1] : J.col[0][1];
    a.key0 = J.key0;
    a.key1 = J.key1;
    a.t = t;
    a.acc = J.acc + (uint64_t)slot * kSlotWords;
    return a;
}

__global__ void __launch_bounds__(kTileBlock) k_batch_tile(const BatchJob* __restrict__ jobs,
                                                           const uint32_t* __restrict__ dyn,
                                                           const BatchWG* __restrict__ wgs,
                                                           const uint32_t* __restrict__ meta, uint32_t m)
{
    __shared__ tilek::TileLds<kTileIpt, kTileBlock> lds;
    if (blockIdx.x >= meta[0]) return;  // whole workgroup
    const BatchWG w = wgs[meta[1] + blockIdx.x];
    const uint32_t* dj = dyn + kDynWords * w.job;
    const uint32_t s0 = m * kBatchTileSweeps;
    if (s0 >= dj[2]) return;  // whole workgroup: no sweep left for this job in this call
    const uint32_t n = min(kBatchTileSweeps, dj[2] - s0);
    const BatchJob& J = jobs[w.job];
    const uint32_t copy = (dj[3] + m) & 1u;
    const SweepArgs a = job_args(J, copy, dj[0] + s0, dj[1] + s0);
    uint8_t* const d0 = copy ? J.col[0][0] : J.col[1][0];
    uint8_t* const d1 = copy ? J.col[0][1] : J.col[1][1];
    const TileGeom tg = *reinterpret_cast<const TileGeom*>(J.rg_words);
    const uint32_t kind = J.cls >> 5;
    if (kind == KIND_ISING_HALF)
        tilek::tile_run<KIND_ISING_HALF, 2, kTileIpt>(a, tg, w.item_base, n, d0, d1, J.table, lds);
    else if (kind == KIND_ISING_ONE)
        tilek::tile_run<KIND_ISING_ONE, 2, kTileIpt>(a, tg, w.item_base, n, d0, d1, J.table, lds);
    else if (kind == KIND_NE)
        tilek::tile_run<KIND_NE, 2, kTileIpt>(a, tg, w.item_base, n, d0, d1, J.table, lds);
    else
        tilek::tile_run<KIND_NE_COUPLED, 2, kTileIpt>(a, tg, w.item_base, n, d0, d1, J.table, lds);
}

__global__ void __launch_bounds__(kBatchPlaneBlock) k_batch_plane(const BatchJob* __restrict__ jobs,
                                                                  const uint32_t* __restrict__ dyn,
                                                                  const BatchWG* __restrict__ wgs,
                                                                  const uint32_t* __restrict__ meta, uint32_t m)
{
    __shared__ planek::PlaneLds<1, kBatchPlaneBlock> lds;
    if (blockIdx.x >= meta[0]) return;  // whole workgroup
    const BatchWG w = wgs[meta[1] + blockIdx.x];
    const uint32_t* dj = dyn + kDynWords * w.job;
    if (m >= dj[2]) return;  // whole workgroup
    const BatchJob& J = jobs[w.job];
    const uint32_t copy = (dj[3] + m) & 1u;
    const SweepArgs a = job_args(J, copy, dj[0] + m, dj[1] + m);
    uint8_t* const d0 = copy ? J.col[0][0] : J.col[1][0];
    uint8_t* const d1 = copy ? J.col[0][1] : J.col[1][1];
    const PlaneGeom pg = *reinterpret_cast<const PlaneGeom*>(J.rg_words);
    const uint32_t ty = w.item_base & 0xFFu, z0 = (w.item_base >> 8) & 0xFFFu, zn = w.item_base >> 20;
    int32_t v[kQ];
    if (J.cls >> 5 == KIND_ISING_HALF) planek::plane_run<KIND_ISING_HALF, 1>(a, pg, ty, z0, zn, d0, d1, J.table, lds, v);
    else planek::plane_run<KIND_ISING_ONE, 1>(a, pg, ty, z0, zn, d0, d1, J.table, lds, v);
    block_accumulate(v[0], v[1], v[2], v[3], a.acc);
}

// One workgroup per job: all of the job's sweeps of this call.
__global__ void __launch_bounds__(kWholeBlock) k_batch_whole(const BatchJob* __restrict__ jobs,
                                                             const uint32_t* __restrict__ dyn,
                                                             const uint32_t* __restrict__ list)
{
    __shared__ tilek::TileLds<kWholeIpt, kWholeBlock> lds;
    const uint32_t j = list[blockIdx.x];
    const uint32_t* dj = dyn + kDynWords * j;
    const uint32_t n = dj[2];
    if (n == 0) return;
    const BatchJob& J = jobs[j];
    const SweepArgs a = job_args(J, 0u, dj[0], dj[1]);
    const TileGeom tg = *reinterpret_cast<const TileGeom*>(J.rg_words);
    const uint32_t kind = J.cls >> 5;
    uint8_t *const d0 = J.col[0][0], *const d1 = J.col[0][1];
    if (kind == KIND_ISING_HALF) {
        if (J.dim == 3) tilek::tile_run<KIND_ISING_HALF, 3, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
        else tilek::tile_run<KIND_ISING_HALF, 2, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
    } else if (kind == KIND_ISING_ONE) {
        if (J.dim == 3) tilek::tile_run<KIND_ISING_ONE, 3, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
        else tilek::tile_run<KIND_ISING_ONE, 2, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
    } else if (kind == KIND_NE) {
        tilek::tile_run<KIND_NE, 2, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
    } else {
        tilek::tile_run<KIND_NE_COUPLED, 2, kWholeIpt>(a, tg, 0u, n, d0, d1, J.table, lds);
    }
}

template <class G>
void store_geom(RowGeomHost& out, const G& g, uint32_t variant, uint32_t copies, uint32_t nitems)
{
    static_assert(sizeof(G) <= sizeof(out.bytes), "geometry storage");
    out = RowGeomHost{};
    __builtin_memcpy(out.bytes, &g, sizeof(G));
    out.variant = variant;
    out.copies = copies;
    out.nitems = nitems;
    out.items_per_wg = 1;
    out.words = g.nitems;
}

}  // namespace

bool batch_tiled_geom(const Geom& g, bool allow_whole, bool allow_tiles, RowGeomHost& out)
{
    TileGeom t;
    const TilePlan whole = whole_plan(g);
    if (allow_whole && tile_geom(g, whole, whole.k, t, kWholeBlock * kWholeIpt)) {
        store_geom(out, t, kBvWhole, 1, 1);
        return true;
    }
    if (!allow_tiles) return false;
    if (g.dim == 2) {
        // the tile with the fewest words updated per launch, its ragged ends
        // filled up to whole waves
        double best = 1e300;
        TileGeom bt{};
        for (uint32_t W : {g.Lh / 4, 8u, 16u, 32u})
            for (uint32_t nty = 1; nty <= g.L; ++nty) {
                const uint32_t H = (g.L + nty - 1) / nty;
                if (W > g.Lh / 4 || H < 8) break;
                if (!tile_geom(g, TilePlan{W, H, 1, kBatchTileSweeps}, kBatchTileSweeps, t, kTileBlock * kTileIpt))
                    continue;
                const double tiles = (double)t.ntx * t.nty;
                double cost = 0;
                for (uint32_t j = 0; j < 2 * kBatchTileSweeps; ++j) cost += (double)tile_words(t, j) + 64.0 * tiles;
                if (cost < best) {
                    best = cost;
                    bt = t;
                }
                break;  // lower tiles only add halos
            }
        if (best == 1e300) return false;
        store_geom(out, bt, kBvTile, 2, bt.ntx * bt.nty);
        return true;
    }
    // 3D: as few columns as fit; the planes of a column are chosen per call
    for (uint32_t nty = 1; nty < 256; ++nty) {
        const uint32_t H = (g.L + nty - 1) / nty;
        PlaneGeom p;
        if (H < 4) break;
        if (g.L >= 4096 || !plane_geom(g, H, g.L, p, kBatchPlaneBlock)) continue;
        store_geom(out, p, kBvPlane, 2, p.nty * g.L);
        return true;
    }
    return false;
}

hipError_t launch_batch_tiled(int family, const BatchJob* jobs, const uint32_t* dyn, const BatchWG* wgs,
                              const uint32_t* meta, uint32_t grid, uint32_t m, hipStream_t s)
{
    if (grid == 0) return hipSuccess;
    if (family == 4)
        hipLaunchKernelGGL(k_batch_tile, dim3(grid), dim3(kTileBlock), 0, s, jobs, dyn, wgs, meta + 2 * family, m);
    else
        hipLaunchKernelGGL(k_batch_plane, dim3(grid), dim3(kBatchPlaneBlock), 0, s, jobs, dyn, wgs, meta + 2 * family,
                           m);
    return hipGetLastError();
}

hipError_t launch_batch_whole(const BatchJob* jobs, const uint32_t* dyn, const uint32_t* list, uint32_t njobs,
                              hipStream_t s)
{
    if (njobs == 0) return hipSuccess;
    hipLaunchKernelGGL(k_batch_whole, dim3(njobs), dim3(kWholeBlock), 0, s, jobs, dyn, list);
    return hipGetLastError();
}

}  // namespace spinlat
