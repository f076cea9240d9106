// kernels_tile.hip -- host side of the tile kernels (tile_device.hpp): tile
// geometry, the choice of tile and sweeps per launch, and the launch.
#include "tile_kernels.h"

namespace spinlat {

namespace {

uint32_t cdiv(uint32_t a, uint32_t b) { return (a + b - 1) / b; }

uint32_t magic(uint32_t d) { return (uint32_t)(((1ull << 32) + d - 1) / d); }

// Launch cost model in us, fitted to 700 timings on MI355X (10% rms).  A launch
// costs `launch`; a CU runs its tiles as many at a time as their threads and
// registers allow, each such round costs `load` (loads, tables, records), and
// a half-sweep costs step + word per wave of words that a SIMD updates, where
// a tile's (3D: a plane's) ragged ends count as `edge` waves.  It puts 2D L =
// 512 (tiles of 8 x 16, 12 sweeps a launch) at 1.31 us per sweep (measured
// 1.34), L = 1048 (16 x 64, 8) at 2.52 (2.54), 3D L = 64 (4 x 4 rows, 3) at
// 2.98 (2.95) and L = 128 (8 x 8 rows, 2) at 5.86 (6.10).
struct Cost {
    double launch, load, step, word, edge;
    uint32_t waves[3];  // waves per SIMD that the registers allow, by words per thread 1, 2, 4
};

const Cost& cost_of(int kind, uint32_t dim, bool coupled)
{
    static const Cost half2 = {3.3, 0.85, 0.166, 0.127, 1.4, {8, 8, 5}}, one2 = {2.85, 1.7, 0.15, 0.217, 0.94, {8, 6, 4}};
    static const Cost ne = {2.6, 1.2, 0.21, 0.135, 0.9, {8, 8, 5}}, nec = {3.2, 1.0, 0.06, 0.166, 0.8, {8, 8, 5}};
    static const Cost half3 = {1.45, 2.04, 0.256, 0.224, 0.17, {8, 7, 4}}, one3 = {1.0, 2.5, 0.24, 0.33, 0.23, {8, 6, 4}};
    if (kind == KIND_ISING_HALF) return dim == 3 ? half3 : half2;
    if (kind == KIND_ISING_ONE) return dim == 3 ? one3 : one2;
    return coupled ? nec : ne;
}

double plan_cost(const TileGeom& t, uint32_t k, const Cost& c)
{
    // rows and planes updated, in the middle of the launch
    const uint32_t cut = 2 * k + 1;
    const double ry = t.wrapy ? t.RY : t.RY - cut, rz = t.wrapz ? t.RZ : t.RZ - cut;
    const double waves = rz * (ry * t.P / 64.0 + c.edge);
    const uint32_t per_cu = (t.ntx * t.nty * t.ntz + 255) / 256;
    const uint32_t regs = c.waves[t.ipt == 1 ? 0 : t.ipt == 2 ? 1 : 2] * 256 / t.block;
    const uint32_t fit = regs < 2048 / t.block ? regs : 2048 / t.block;
    const uint32_t at_once = per_cu < fit ? per_cu : fit ? fit : 1;
    const double rounds = (double)((per_cu + at_once - 1) / at_once);
    return c.launch + rounds * (c.load + 2.0 * k * (c.step + c.word * at_once * waves / 4.0));
}

// The same for tiles on bit words at c = 0.1: every word costs its load and store,
// and a half-sweep is mostly latency (within 5% of 20 timings, L = 1048 .. 4096).
double bits_cost(const TileGeom& t, uint32_t k)
{
    const uint32_t per_cu = (t.ntx * t.nty + 255) / 256, fit = t.ipt == 1 ? 2048 / t.block : 2;
    const uint32_t at_once = per_cu < fit ? per_cu : fit;
    const double rounds = (double)((per_cu + at_once - 1) / at_once);
    const double held = at_once * ((t.nitems + 63) / 64), updated = at_once * (t.P / 8) * (t.RY - 2.0 * k) / 64.0;
    return 1.0 + rounds * (0.26 * held + 2.0 * k * (0.85 + 0.0235 * updated));
}

}  // namespace

TilePlan whole_plan(const Geom& g) { return TilePlan{g.Lh / 4, g.L, g.L, kTileWhole}; }

bool tile_geom(const Geom& g, const TilePlan& p, uint32_t k, TileGeom& t, uint32_t max_items)
{
    t = TileGeom{};
    t.L = g.L;
    t.ncols = g.Lh / 4;
    t.W = p.W < t.ncols ? p.W : t.ncols;
    t.H = p.H < g.L ? p.H : g.L;
    t.Z = g.dim == 3 ? (p.Z < g.L ? p.Z : g.L) : 1;
    if (!t.W || !t.H || !t.Z || !k) return false;
    t.bits = p.bits;
    t.wrapx = !t.bits && t.W == t.ncols;
    t.wrapy = t.H == g.L;
    t.wrapz = g.dim == 2 || t.Z == g.L;
    // a half-sweep needs one more site on each side: 2 k rows and planes, and
    // 2 k sites of the 8 that a word pair covers in x
    t.hx = t.bits ? 8 : t.wrapx ? 0 : cdiv(2 * k, 8);
    t.hy = t.wrapy ? 0 : 2 * k;
    t.hz = t.wrapz ? 0 : 2 * k;
    if (t.W + t.hx > t.ncols || t.H + t.hy > t.L || (g.dim == 3 && t.Z + t.hz > t.L)) return false;
    t.P = t.W + 2 * t.hx;
    t.RY = t.H + 2 * t.hy;
    t.RZ = t.Z + 2 * t.hz;
    const uint32_t words = t.bits ? t.P / 8 : t.P;  // of a row
    const uint64_t n = (uint64_t)words * t.RY * t.RZ;
    if (n > max_items || (t.bits && (t.wrapy || 2 * k > 32 || t.W % 8 != 0 || n > 2048))) return false;
    t.nitems = (uint32_t)n;
    t.ntx = cdiv(t.ncols, t.W);
    t.nty = cdiv(t.L, t.H);
    t.ntz = g.dim == 3 ? cdiv(t.L, t.Z) : 1;
    t.magicP = magic(words);
    t.magicRY = magic(t.RY);
    t.ipt = t.nitems <= 1024 ? 1 : t.nitems <= 2048 ? 2 : 4;
    t.block = cdiv(cdiv(t.nitems, t.ipt), 64) * 64;
    return true;
}

uint64_t tile_words(const TileGeom& t, uint32_t j)
{
    const uint32_t cut = 2 * (j + 1);
    const uint64_t ry = t.wrapy ? t.RY : t.RY - cut, rz = t.wrapz ? t.RZ : t.RZ - cut;
    return ry * rz * t.P * t.ntx * t.nty * t.ntz;
}

// Large North-East lattices with J = 0 where an up-flip draws, not a down-flip (c <=
// 1/2), so that few groups draw: tiles of bit words (kernels_tile_bits.hip).  us per
// sweep, 4-site words against bits: L = 1536, c = 0.1 4.05 and 2.26; 1800, c = 0.3
// 4.3 and 3.6; 4096 13.6 and 3.5 (c = 0.3 6.3), 8192, rows otherwise, 48 and 12; but
// 1304, c = 0.3 2.6 and 3.2, and 4096, c = 0.7 13.7 and 15.2.
static TilePlan bits_plan(const Geom& g, const TilePlan& other)
{
    TilePlan best = other;
    TileGeom t;
    double best_us = 1e30;
    for (uint32_t k : {4u, 6u, 8u, 12u})
        for (uint32_t W : {16u, 32u, 64u, 128u})
            for (uint32_t H : {16u, 32u, 64u, 128u}) {
                TilePlan p{W, H, 1, k};
                p.bits = 1;
                if (!tile_geom(g, p, k, t)) continue;
                const double us = bits_cost(t, k) / k;
                if (us < best_us) {
                    best_us = us;
                    best = p;
                }
            }
    return best;
}

TilePlan tile_plan(const Geom& g, int kind, bool coupled, bool sparse)
{
    const Cost& c = cost_of(kind, g.dim, coupled);
    TilePlan best{};
    TileGeom t;
    double best_us = 1e30;
    const TilePlan whole = whole_plan(g);
    if (tile_geom(g, whole, whole.k, t)) {  // no launch cost to speak of
        best = whole;
        best_us = 2.0 * (c.step + c.word * (t.nitems / 64.0 + c.edge) / 4.0);
    }
    // several rounds of tiles per CU: 16 words x 64 rows and 4 sweeps, which
    // leaves two workgroups of 12 waves on a CU, was fastest at every size
    // (spin-1/2 L = 4096: 12.6 against 14-16 for the other shapes of 4 sweeps,
    // 16 and more with 2 or 3; L = 3000: 8.4 against 11-12)
    const TilePlan large{16, 64, 1, 4};
    if (g.dim == 2 && tile_geom(g, large, large.k, t)) {
        if (sparse && kind == KIND_NE && !coupled && t.ntx * t.nty > 256) return bits_plan(g, large);
        if (t.ntx * t.nty > 2 * 256) return large;
    }
    for (uint32_t k : {1u, 2u, 3u, 4u, 6u, 8u, 12u})
        for (uint32_t W : {4u, 8u, 16u, 32u, 64u})
            for (uint32_t H : {2u, 4u, 8u, 16u, 32u, 64u, 128u})
                for (uint32_t Z : {1u, 2u, 4u, 8u, 16u}) {
                    // 3D tiles hold whole rows
                    if (g.dim == 2 ? Z > 1 || W > g.Lh / 4 : W < 64) break;
                    const TilePlan p{g.dim == 2 ? W : g.Lh / 4, H, Z, k};
                    if (!tile_geom(g, p, k, t)) continue;
                    const double us = plan_cost(t, k, c) / k;
                    if (us < best_us) {
                        best_us = us;
                        best = p;
                    }
                }
    return best;
}

hipError_t launch_tile(const SweepArgs& a, int kind, const TileGeom& tg, uint32_t k, uint8_t* dst0, uint8_t* dst1,
                       hipStream_t s)
{
    if (tg.bits) return launch_tile_bits(a, tg, k, dst0, dst1, s);
    if (kind == KIND_ISING_HALF) return launch_tile_half(a, tg, k, dst0, dst1, s);
    if (kind == KIND_ISING_ONE) return launch_tile_one(a, tg, k, dst0, dst1, s);
    return launch_tile_ne(a, tg, k, dst0, dst1, s);
}

}  // namespace spinlat
