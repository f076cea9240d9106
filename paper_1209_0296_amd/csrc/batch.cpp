// batch.cpp -- host side of the batch ABI (include/spinlat.h, "Batches").
//
// The caller's arena holds, in order: the device job table, two sets of
// per-call upload areas (per-job counters {t, record slot, sweeps in this call,
// current copy}, the work list in one segment per kernel family, the count and
// offset of each segment and the list of resident jobs; calls alternate
// between the two sets), the fold table and
// buffer for record readback, and a heap from which each job's lattice (two
// colour arrays, or two copies of them for fused jobs) and record ring are
// carved first-fit.  Admission by footprint is the heap allocation succeeding.
// Tiles and walks along z need a second lattice copy, lent from the heap's free
// ranges; where there is no room for it, or a new job takes it, a job runs in the
// one-copy class that sl_batch_job_bytes reports, until room comes free again.
//
// A call (sl_batch_sweep) uploads the counters and work lists from pinned
// staging (double-buffered, so the host never waits for the previous call),
// runs the resident jobs' launch on a second stream of the library's own
// while the per-sweep launches of the other jobs run on the caller's stream,
// and joins the two.  The per-sweep launches of the kernel families are
// captured once per (sweeps, grid buckets) shape into HIP graphs, each on one
// stream, and replayed; the kernels read the true segment counts from device
// memory.  The families of 3D jobs run on a third stream of the library's,
// beside the other families (they touch disjoint jobs), so that one family's
// waves fill the issue slots another leaves idle.  Workgroups of tiles and
// columns are listed heaviest first and left in the hardware's order over the
// XCDs: a contiguous range per XCD, good for one lattice, put the large jobs of
// a mix on few of them (256 served jobs: 50.7 ms so, 46.1 spread, 43.6 sorted).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/spinlat.h"
#include "batch_internal.h"
#include "host_common.h"
#include "plane_plan.h"
#include "spinlat_internal.h"

using namespace spinlat;
using namespace spinlat::host;

namespace {

constexpr uint64_t kDefaultMaxWG = 1ull << 20;
constexpr size_t kGraphCache = 16;

uint64_t max_wg(const sl_batch_config* c) { return c->max_workgroups ? c->max_workgroups : kDefaultMaxWG; }

// One set of per-call device upload areas.
struct UploadLayout {
    size_t dyn, wgs, counts, res;  // offsets from the set's start
    size_t bytes;
};

UploadLayout upload_layout(const sl_batch_config* c)
{
    UploadLayout u{};
    size_t off = 0;
    u.dyn = off;
    off += round_up((size_t)c->max_jobs * kDynWords * sizeof(uint32_t), kAlign);
    u.wgs = off;
    off += round_up((size_t)max_wg(c) * sizeof(BatchWG), kAlign);
    u.counts = off;
    off += kAlign;
    u.res = off;
    off += round_up((size_t)c->max_jobs * sizeof(uint32_t), kAlign);
    u.bytes = off;
    return u;
}

struct BaseLayout {
    size_t jobs, up[2], foldtab, fold, heap;
    UploadLayout u;
};

BaseLayout base_layout(const sl_batch_config* c)
{
    BaseLayout b{};
    b.u = upload_layout(c);
    size_t off = 0;
    b.jobs = off;
    off += round_up((size_t)c->max_jobs * sizeof(BatchJob), kAlign);
    for (int k = 0; k < 2; ++k) {
        b.up[k] = off;
        off += b.u.bytes;
    }
    b.foldtab = off;
    off += round_up((size_t)c->max_jobs * sizeof(BatchFold), kAlign);
    b.fold = off;  // every job's unread records at once
    off += round_up((size_t)c->max_jobs * c->record_capacity * kRecordWords * sizeof(int64_t), kAlign);
    b.heap = off;
    return b;
}

sl_status check_config(const sl_batch_config* c)
{
    if (!c) return fail(SL_E_INVALID, "config is NULL");
    if (c->abi_version != SL_ABI_VERSION)
        return fail(SL_E_INVALID, "abi_version %u != %u", c->abi_version, SL_ABI_VERSION);
    if (c->max_jobs < 1 || c->max_jobs > (1u << 24)) return fail(SL_E_INVALID, "max_jobs out of range");
    if (c->record_capacity < 2) return fail(SL_E_INVALID, "record_capacity must be >= 2");
    if (c->tile_rows < 0) return fail(SL_E_INVALID, "tile_rows must be >= 0");
    if (c->flags & ~(uint32_t)(SL_BATCH_NO_GRAPH | SL_BATCH_NO_FUSED | SL_BATCH_NO_RESIDENT))
        return fail(SL_E_INVALID, "unknown batch flags 0x%x", c->flags);
    return SL_OK;
}

struct JobFoot {
    uint64_t nh;
    size_t col_bytes, ring_bytes, total;
};

JobFoot job_foot(const sl_params* p, uint32_t cap, uint32_t copies)
{
    JobFoot f{};
    const uint64_t nsites = p->dim == 2 ? (uint64_t)p->L * p->L : (uint64_t)p->L * p->L * p->L;
    f.nh = nsites / 2;
    f.col_bytes = round_up(f.nh, kAlign);
    f.ring_bytes = round_up((size_t)cap * kSlotWords * sizeof(int64_t), kAlign);
    f.total = 2 * copies * f.col_bytes + f.ring_bytes;
    return f;
}

int default_rows(int dim, bool fused) { return fused ? 4 : dim == 3 ? 4 : 8; }

struct JobHost {
    bool used = false;
    sl_params params{};
    int kind = 0;
    size_t off = 0;
    JobFoot foot{};
    // class in use; the one the footprint is for; the one to use while there is room
    RowGeomHost geom{}, least{}, want{};
    bool lent = false;            // copy 1 lies at off2, in a free range of the heap
    bool kept = false;            // copy 1 lies at off2, in a block of its own
    size_t off2 = 0;
    uint32_t cur = 0;  // copy holding the current state (fused jobs alternate)
    uint64_t t = 0, remaining = 0, pending = 0, first_t = 0, done = 0;
    uint64_t table[kMaxLut] = {};
    size_t table_n = 0;
};

bool resident_job(const JobHost& J) { return J.geom.variant == kBvResident || J.geom.variant == kBvWhole; }

// Kernel kind of a job's class: the model kind, with coupled NE jobs apart.
int class_kind(const JobHost& J)
{
    return J.params.model == SL_NE_COUPLED ? kBatchKindNeCoupled : J.kind;
}

// Workgroups of a job in a call, at most.
uint64_t most_workgroups(const RowGeomHost& g)
{
    if (g.variant == kBvResident || g.variant == kBvWhole) return 0;  // not in the work list
    const uint64_t per = g.variant == kBvPlane ? 4 : g.items_per_wg;
    return (g.nitems + per - 1) / per;
}

// Launches that `sweeps` sweeps in class g take if each leaves the state in the
// other of two copies.
uint64_t copy_flips(const RowGeomHost& g, uint64_t sweeps)
{
    if (g.variant == kBvTile) return family_launches(4, sweeps);
    return g.copies == 2 ? sweeps : 0;
}

// Classes of whole 2D rows.
bool row_class(uint32_t variant)
{
    return variant <= kBvWalkD1 || (variant >= kBvFusedD4 && variant <= kBvFusedD1);
}

// Can a job on tiles run a call in its row class, at no more workgroups?
bool has_rows(const JobHost& J)
{
    return J.geom.variant == kBvTile && row_class(J.least.variant) &&
           most_workgroups(J.least) <= most_workgroups(J.geom);
}

// Does a job on tiles run a call of n sweeps on its rows, when such jobs have
// `sites` sites in all?  A tile's halo and start are paid per launch of up to four
// sweeps, so where the chip is full, rows are faster for few sweeps, and for spin-1/2
// whenever the last launch has fewer (us a call, rows against tiles: 16 jobs of L = 1024,
// 2^24 sites: spin-1/2 n = 1 40 and 45, 2 54 and 53; of L = 1536 1 59 and 84, 2 94 and 102, 3
// 132 and 125; 64 of L = 1024: spin-1/2 1 85 and 117, 2 132 and 148, 3 179 and 189, 5 275 and
// 308, 64 3172 and 3086; spin-1 1 116 and 137, 2 198 and 197, 3 279 and 266; North-East 1 93
// and 122, 2 152 and 158, 3 211 and 201).
bool runs_on_rows(const JobHost& J, uint64_t n, uint64_t sites)
{
    const bool half = class_kind(J) == KIND_ISING_HALF;
    if (n == 1) return sites >= (1ull << 24);
    if (class_kind(J) == KIND_ISING_ONE) return false;
    if (n == 2) return sites >= (half ? 1ull << 25 : 1ull << 26);
    return half && n % kBatchTileSweeps != 0 && n < 32 && sites >= (1ull << 26);
}

// Planes of a column of the walks along z, for a call whose jobs have `planes`
// planes of columns in all: about 768 workgroups (three per CU), 4 to 32 planes
// (a column recomputes two colour-0 planes).
uint32_t plane_depth(uint64_t planes)
{
    const uint64_t d = (planes + 767) / 768;
    return (uint32_t)(d < 4 ? 4 : d > 32 ? 32 : d);
}

struct Lent {
    size_t start;
    uint32_t job;
};

struct GraphEntry {
    uint64_t key;  // sweeps * 2 + upload set
    uint32_t grid[kBatchFamilies];
    hipGraphExec_t exec;
};

uint32_t bucket(uint64_t n)
{
    if (n == 0) return 0;
    uint32_t b = 64;
    while (b < n) b <<= 1;
    return b;
}

}  // namespace

struct sl_batch {
    sl_batch_config cfg;
    uint8_t* arena;
    size_t arena_bytes;
    hipStream_t stream;  // the caller's
    hipStream_t side;    // resident jobs run here, concurrently
    hipStream_t par;     // the row-group families run here, beside the others
    hipStream_t cap;     // graph capture only
    hipEvent_t ev_up[2];   // per upload set: its uploads were consumed by the launches
    hipEvent_t ev_fork, ev_join, ev_par;
    BaseLayout base;
    std::vector<JobHost> jobs;
    FreeList heap;       // free ranges of the job heap
    std::map<size_t, Lent> lent;  // lent second copies in free ranges, by their end
    uint64_t list_most;  // workgroups of every job's class in a call, at most
    bool retry;          // room has come free since jobs last went back to their wanted class
    bool refused;        // a job found no room since the last call
    uint8_t* h_up[2];    // pinned upload staging, one per upload set
    sl_record* h_stage;  // pinned [max_jobs * record_capacity]
    BatchFold* h_fold;   // pinned [max_jobs]
    uint64_t calls;
    std::vector<GraphEntry> graphs;
};

namespace {

BatchJob* d_jobs(const sl_batch* b) { return reinterpret_cast<BatchJob*>(b->arena + b->base.jobs); }
uint8_t* d_up(const sl_batch* b, int k) { return b->arena + b->base.up[k]; }

Geom geom_of(const sl_params* p, uint64_t nh)
{
    Geom g;
    g.L = (uint32_t)p->L;
    g.Lh = (uint32_t)(p->L / 2);
    g.dim = (uint32_t)p->dim;
    g.rows = p->dim == 2 ? g.L : g.L * g.L;
    g.nh = nh;
    return g;
}

uint8_t* col_of(const sl_batch* b, const JobHost& J, uint32_t copy, uint32_t colour)
{
    if ((J.lent || J.kept) && copy == 1) return b->arena + J.off2 + colour * J.foot.col_bytes;
    return b->arena + J.off + (2 * copy + colour) * J.foot.col_bytes;
}

unsigned long long* ring_of(const sl_batch* b, uint32_t j)
{
    const JobHost& J = b->jobs[j];
    return reinterpret_cast<unsigned long long*>(b->arena + J.off + 2 * J.least.copies * J.foot.col_bytes);
}

SweepArgs job_args(const sl_batch* b, uint32_t j)
{
    const JobHost& J = b->jobs[j];
    SweepArgs a{};
    a.col[0] = col_of(b, J, J.cur, 0);
    a.col[1] = col_of(b, J, J.cur, 1);
    a.g = geom_of(&J.params, J.foot.nh);
    a.key0 = (uint32_t)J.params.seed;
    a.key1 = (uint32_t)(J.params.seed >> 32);
    a.lut = d_jobs(b)[j].table;
    a.lut_n = (int32_t)J.table_n;
    return a;
}

// Device job-table entry of a job in its present class.
BatchJob job_entry(const sl_batch* b, uint32_t j)
{
    const JobHost& J = b->jobs[j];
    BatchJob entry;
    std::memset(&entry, 0, sizeof(BatchJob));
    for (uint32_t cp = 0; cp < J.geom.copies; ++cp)
        for (uint32_t c = 0; c < 2; ++c) entry.col[cp][c] = col_of(b, J, cp, c);
    entry.acc = ring_of(b, j);
    entry.key0 = (uint32_t)J.params.seed;
    entry.key1 = (uint32_t)(J.params.seed >> 32);
    entry.cls = batch_class(class_kind(J), J.params.dim, J.geom.variant);
    entry.copies = J.geom.copies;
    entry.dim = (uint32_t)J.params.dim;
    entry.table_n = (uint32_t)J.table_n;
    std::memcpy(entry.rg_words, J.geom.bytes, sizeof(entry.rg_words));
    std::memcpy(entry.row_words, J.least.bytes, sizeof(entry.row_words));
    entry.row_cls = batch_class(class_kind(J), J.params.dim, J.least.variant);
    std::memcpy(entry.table, J.table, J.table_n * sizeof(uint64_t));
    return entry;
}

// Tiles and walks along z need a second copy of the lattice, which the footprint
// that callers are told, and by which jobs are admitted, does not hold.  It lies in
// a free range of the heap, as high as possible, without being allocated there: a
// job that is given that range takes it back.  So what fits an arena does not
// depend on the second copies.
bool find_second(const sl_batch* b, size_t bytes, size_t* off)
{
    const std::map<size_t, Lent>& lent = b->lent;
    const std::map<size_t, size_t>& ranges = b->heap.map();
    for (auto r = ranges.rbegin(); r != ranges.rend(); ++r) {
        const size_t start = r->first;
        size_t end = start + r->second;
        for (auto l = lent.upper_bound(end); l != lent.begin();) {
            --l;
            if (l->first <= start || end - l->first >= bytes) break;  // of another range, or a gap
            end = l->second.start;
        }
        if (end - start >= bytes) {
            *off = end - bytes;
            return true;
        }
    }
    return false;
}

// The class that job J, one of the batch's, runs in from here on.
void set_class(sl_batch* b, JobHost& J, const RowGeomHost& geom)
{
    b->list_most = b->list_most - most_workgroups(J.geom) + most_workgroups(geom);
    J.geom = geom;
}

// Device job-table entry of job j in its present class, in stream order: a start of
// no lattice and no ring.
hipError_t write_entry(sl_batch* b, uint32_t j)
{
    const BatchJob entry = job_entry(b, j);
    StartArgs s{};
    s.blob_dst = reinterpret_cast<uint32_t*>(d_jobs(b) + j);
    s.blob_words = (uint32_t)(sizeof(BatchJob) / 4);
    StartBlob blob;
    std::memcpy(blob.w, &entry, sizeof(BatchJob));
    return launch_start(s, b->jobs[j].kind, blob, b->stream);
}

void give_up_second(sl_batch* b, JobHost& J)
{
    if (J.lent) b->lent.erase(J.off2 + 2 * J.foot.col_bytes);
    if (J.kept) b->heap.release(J.off2, 2 * J.foot.col_bytes);
    J.lent = J.kept = false;
}

// Job j goes on in its least class: the state moves to the first copy, a second one
// apart from it is given up.
hipError_t demote(sl_batch* b, uint32_t j)
{
    JobHost& J = b->jobs[j];
    const bool apart = J.lent || J.kept;  // copy 1
    if (apart && J.cur == 1) {
        const hipError_t e = hipMemcpyAsync(col_of(b, J, 0, 0), col_of(b, J, 1, 0), 2 * J.foot.col_bytes,
                                            hipMemcpyDeviceToDevice, b->stream);
        if (e != hipSuccess) return e;
    }
    if (apart) J.cur = 0;
    give_up_second(b, J);
    set_class(b, J, J.least);
    return write_entry(b, j);
}

// Lent second copies in [off, off + bytes): their jobs.
std::vector<uint32_t> lent_in(const sl_batch* b, size_t off, size_t bytes)
{
    std::vector<uint32_t> out;
    for (auto l = b->lent.upper_bound(off); l != b->lent.end() && l->second.start < off + bytes; ++l)
        out.push_back(l->second.job);
    return out;
}

// These are given up: their jobs go on in the class that needs one.
hipError_t take_back(sl_batch* b, size_t off, size_t bytes)
{
    for (uint32_t j : lent_in(b, off, bytes)) {
        const hipError_t e = demote(b, j);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Tiles of 2D rows that a row class takes in few strips need more workgroups than
// it (L = 1536: 276 and 96).  Jobs whose least classes fit the work list must not
// overflow it, so where `more` further workgroups would, jobs leave their tiles,
// those that save most first.
hipError_t make_list_room(sl_batch* b, uint64_t more)
{
    const uint64_t most = max_wg(&b->cfg);
    if (b->list_most + more <= most) return hipSuccess;
    std::vector<std::pair<uint64_t, uint32_t>> saves;
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        const JobHost& J = b->jobs[j];
        if (J.used && most_workgroups(J.geom) > most_workgroups(J.least))
            saves.emplace_back(most_workgroups(J.geom) - most_workgroups(J.least), j);
    }
    std::sort(saves.rbegin(), saves.rend());
    for (size_t i = 0; i < saves.size() && b->list_most + more > most; ++i) {
        const hipError_t e = demote(b, saves[i].second);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// A second copy for a job in its wanted class, where that needs one.
bool lend_second(sl_batch* b, uint32_t j, JobHost& J)
{
    if (J.want.copies <= J.least.copies) return true;
    J.lent = find_second(b, 2 * J.foot.col_bytes, &J.off2);
    if (J.lent) b->lent[J.off2 + 2 * J.foot.col_bytes] = Lent{J.off2, j};
    return J.lent;
}

// Jobs that gave up their tiles or walks take them again where room has come free
// since, in the order of their slots.  Not while jobs are refused for want of room:
// the next one would take the copies back at once.
hipError_t promote(sl_batch* b)
{
    const bool refused = b->refused;
    b->refused = false;
    if (!b->retry || refused) return hipSuccess;
    b->retry = false;
    size_t none = ~(size_t)0;  // the least second copy that found no room
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        JobHost& J = b->jobs[j];
        if (!J.used || !J.remaining || J.geom.variant == J.want.variant) continue;
        const uint64_t now = most_workgroups(J.geom), then = most_workgroups(J.want);
        const size_t second = 2 * J.foot.col_bytes;
        if (then > now && b->list_most - now + then > max_wg(&b->cfg)) continue;
        if (J.want.copies > J.least.copies && second >= none) continue;
        if (!lend_second(b, j, J)) {
            none = second;
            continue;
        }
        set_class(b, J, J.want);  // J.cur: 0 in a class of one copy, else either way
        const hipError_t e = write_entry(b, j);
        if (e != hipSuccess) {
            give_up_second(b, J);
            set_class(b, J, J.least);
            return e;
        }
    }
    return hipSuccess;
}

sl_status check_job(const sl_batch* b, uint32_t j)
{
    if (!b) return fail(SL_E_INVALID, "NULL batch");
    if (j >= b->jobs.size() || !b->jobs[j].used) return fail(SL_E_INVALID, "no job %u", j);
    return SL_OK;
}

// Parameters of a job (record capacity from the batch), its class and footprint.
// geom is the class to use, least the one while the arena has no room for a second
// lattice copy (foot: the footprint of least).
sl_status prepare_job(const sl_batch_config* cfg, const sl_params* params, sl_params* p, JobFoot* foot,
                      RowGeomHost* geom, RowGeomHost* least, uint64_t* table, size_t* table_n)
{
    if (!params) return fail(SL_E_INVALID, "params is NULL");
    *p = *params;
    p->record_capacity = cfg->record_capacity;
    sl_status st = validate(p);
    if (st != SL_OK) return st;
    if (is_sub_lattice(p->model))
        return fail(SL_E_UNSUPPORTED, "batched jobs use the checkerboard sweep; the NE "
                                      "sub-lattice algorithm runs as a single lattice");
    *table_n = build_table(p, table);
    bool lut32 = true;
    for (size_t i = 0; i < *table_n; ++i)
        if (table[i] == 0) lut32 = false;
    const bool coupled = p->model == SL_NE_COUPLED;
    const bool spin_half_table = kind_of(p) == KIND_ISING_HALF || coupled;
    const uint64_t nh = (p->dim == 2 ? (uint64_t)p->L * p->L : (uint64_t)p->L * p->L * p->L) / 2;
    const Geom g = geom_of(p, nh);
    const bool fused = p->dim == 2 && !(cfg->flags & SL_BATCH_NO_FUSED);
    const int H = cfg->tile_rows > 0 ? cfg->tile_rows : default_rows(p->dim, fused);
    if (!(cfg->flags & SL_BATCH_NO_RESIDENT) && batch_resident_geom(g, *least)) {
        // resident jobs run the direct update in LDS: any table
    } else if (!batch_geom(g, H, lut32 || !spin_half_table, fused, *least)) {
        return fail(SL_E_UNSUPPORTED, "L = %d does not fit the batched kernels", p->L);
    }
    if (coupled && least->variant == kBvWindow)
        return fail(SL_E_UNSUPPORTED, "batched coupled NE jobs need a colour row that fits one wave "
                                      "and every threshold >= 1 (L = %d), or a lattice that fits LDS", p->L);
    *foot = job_foot(p, cfg->record_capacity, least->copies);
    // tiles and walks along z, unless the caller asked for a strip height or for
    // fewer workgroups than they take; nor rows that fill the waves of the other
    // classes: 3D row groups, and 2D walks in a batch that can fill the chip (64 jobs
    // of L = 2048, 64 lanes, walks against tiles: spin-1/2 174 and 188, spin-1 246 and
    // 284, NE 186 and 195; of L = 1536, 48 lanes, 122 and 114; 8 jobs of L = 2048 32 and
    // 26)
    const bool fills = p->dim == 2 && p->L >= 1792 && least->variant == kBvWalkD4 &&
                       (uint64_t)cfg->max_jobs * nh > (1ull << 26);
    const bool rows = least->variant == kBvRowsD4 && rows_beat_plane(g, kind_of(p), 8192);
    if (fills || rows || !(p->model == SL_NORTH_EAST || lut32) ||
        !batch_tiled_geom(g, !(cfg->flags & SL_BATCH_NO_RESIDENT),
                          !(cfg->flags & SL_BATCH_NO_FUSED) && cfg->tile_rows == 0, *geom) ||
        (cfg->max_workgroups && most_workgroups(*geom) > most_workgroups(*least)))
        *geom = *least;
    return SL_OK;
}

// Launches of one kernel family for n sweeps: the tiles once per
// kBatchTileSweeps sweeps, fused jobs and walks along z once per sweep, the
// others once per colour.
hipError_t enqueue_family(sl_batch* b, int k, int f, uint64_t n, uint32_t grid, hipStream_t s)
{
    const UploadLayout& u = b->base.u;
    const uint32_t* dyn = reinterpret_cast<const uint32_t*>(d_up(b, k) + u.dyn);
    const BatchWG* wgs = reinterpret_cast<const BatchWG*>(d_up(b, k) + u.wgs);
    const uint32_t* meta = reinterpret_cast<const uint32_t*>(d_up(b, k) + u.counts);
    hipError_t e = hipSuccess;
    if (f == 4 || f == 5) {
        for (uint64_t m = 0; m < family_launches(f, n) && e == hipSuccess && grid; ++m)
            e = launch_batch_tiled(f, d_jobs(b), dyn, wgs, meta, grid, (uint32_t)m, s);
        return e;
    }
    for (uint64_t s2 = 0; s2 < n && e == hipSuccess && grid; ++s2)
        for (uint32_t c = 0; c < (f == 2 ? 1u : 2u) && e == hipSuccess; ++c)
            e = launch_batch_family(f, d_jobs(b), dyn, wgs, meta, grid, c, (uint32_t)s2, s);
    return e;
}

// The per-sweep launches of the shape (n, grids) on upload set k as a graph,
// captured on first use.
sl_status graph_for(sl_batch* b, int k, uint64_t n, const uint32_t (&grid)[kBatchFamilies], hipGraphExec_t* out)
{
    const uint64_t key = n * 2 + (uint64_t)k;
    for (size_t i = 0; i < b->graphs.size(); ++i)
        if (b->graphs[i].key == key && std::equal(grid, grid + kBatchFamilies, b->graphs[i].grid)) {
            // most recently used last: eviction takes the front
            const GraphEntry g = b->graphs[i];
            b->graphs.erase(b->graphs.begin() + (long)i);
            b->graphs.push_back(g);
            *out = g.exec;
            return SL_OK;
        }
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_fail(e, "batch: begin graph capture");
    hipError_t le = hipSuccess;
    for (int f = 0; f < kBatchFamilies && le == hipSuccess; ++f) le = enqueue_family(b, k, f, n, grid[f], b->cap);
    e = hipStreamEndCapture(b->cap, &graph);
    if (le != hipSuccess || e != hipSuccess) {
        if (graph) (void)hipGraphDestroy(graph);
        return hip_fail(le != hipSuccess ? le : e, "batch: graph capture");
    }
    hipGraphExec_t exec = nullptr;
    e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return hip_fail(e, "batch: graph instantiate");
    if (b->graphs.size() >= kGraphCache) {
        // the least recently used graph may still run: wait before destroying
        // it (graphs of earlier calls run on the caller's stream or on par,
        // which the caller's stream joins at the end of every call)
        e = hipStreamSynchronize(b->stream);
        if (e == hipSuccess) e = hipStreamSynchronize(b->par);
        if (e != hipSuccess) return hip_fail(e, "batch: synchronise before graph eviction");
        (void)hipGraphExecDestroy(b->graphs.front().exec);
        b->graphs.erase(b->graphs.begin());
    }
    GraphEntry ge{key, {}, exec};
    std::copy(grid, grid + kBatchFamilies, ge.grid);
    b->graphs.push_back(ge);
    *out = exec;
    return SL_OK;
}

// sl_batch_add, or (keep) sl_batch_add_keeping.
sl_status add_job(sl_batch* b, const sl_params* params, uint64_t sweeps, bool keep, uint32_t* job_id)
{
    if (!b) return fail(SL_E_INVALID, "NULL batch");
    if (!job_id) return fail(SL_E_INVALID, "job_id is NULL");
    JobHost J;
    sl_status st = prepare_job(&b->cfg, params, &J.params, &J.foot, &J.want, &J.least, J.table, &J.table_n);
    if (st != SL_OK) return st;
    J.geom = J.want;
    if (sweeps > (1ull << 32) - J.params.t0)  // validate() keeps t0 < 2^32
        return fail(SL_E_OVERFLOW, "t0 + sweeps would pass 2^32");
    uint32_t j = 0;
    while (j < b->jobs.size() && b->jobs[j].used) ++j;
    if (j == b->jobs.size()) return fail(SL_E_STATE, "job table full (%u jobs)", b->cfg.max_jobs);
    if (!b->heap.alloc(J.foot.total, &J.off)) {
        b->refused = true;
        return fail(SL_E_BUFFER, "arena has no free block of %zu bytes for this job", J.foot.total);
    }
    const bool list_full = b->list_most + most_workgroups(J.want) > max_wg(&b->cfg);
    if (list_full && most_workgroups(J.want) > most_workgroups(J.least)) J.geom = J.least;
    if (keep) {
        // with other jobs in the arena, only beside every copy that they and it want
        const size_t second = 2 * J.foot.col_bytes;
        const bool need = J.want.copies > J.least.copies;
        const bool others = std::any_of(b->jobs.begin(), b->jobs.end(), [](const JobHost& o) { return o.used; });
        bool room = !list_full && lent_in(b, J.off, J.foot.total).empty();
        if (room && need) {
            J.kept = b->heap.alloc(second, &J.off2);
            room = J.kept && lent_in(b, J.off2, second).empty();
        }
        if (!room && others) {
            if (J.kept) b->heap.release(J.off2, second);
            b->heap.release(J.off, J.foot.total);
            b->refused = true;
            return fail(SL_E_BUFFER, "arena has no room for this job beside the jobs' second lattice copies");
        }
        if (need && !J.kept) J.geom = J.least;
    }
    hipError_t e = take_back(b, J.off, J.foot.total);
    if (e == hipSuccess) e = make_list_room(b, most_workgroups(J.geom));
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(b->stream);
        give_up_second(b, J);
        b->heap.release(J.off, J.foot.total);
        return hip_fail(e, "batch add");
    }
    if (!keep && J.geom.variant == J.want.variant && !lend_second(b, j, J)) J.geom = J.least;
    J.used = true;
    J.kind = kind_of(&J.params);
    J.t = J.params.t0;
    J.first_t = J.params.t0;
    J.remaining = sweeps;
    J.cur = 0;
    b->jobs[j] = J;
    b->list_most += most_workgroups(J.geom);

    // device job-table entry, written by the start kernel
    static_assert(sizeof(BatchJob) <= sizeof(StartBlob), "a job entry travels in the start kernel's arguments");
    const BatchJob entry = job_entry(b, j);
    SweepArgs a = job_args(b, j);
    const uint64_t bern = thr_from_prob(J.params.c);
    e = start_lattice(a, &J.params, J.kind, bern, ring_of(b, j), (uint64_t)b->cfg.record_capacity * kSlotWords,
                      d_jobs(b) + j, &entry, sizeof(BatchJob), b->stream);
    // record r_0: observables of the initial state
    a.acc = ring_of(b, j);
    if (e == hipSuccess) e = launch_observe(a, J.kind, b->stream);
    if (e != hipSuccess) {
        (void)hipStreamSynchronize(b->stream);
        b->heap.release(J.off, J.foot.total);
        give_up_second(b, b->jobs[j]);
        b->list_most -= most_workgroups(J.geom);
        b->jobs[j] = JobHost();
        return hip_fail(e, "batch add");
    }
    b->jobs[j].pending = 1;
    *job_id = j;
    return SL_OK;
}

}  // namespace

extern "C" {

sl_status sl_batch_base_bytes(const sl_batch_config* cfg, size_t* bytes)
{
    sl_status st = check_config(cfg);
    if (st != SL_OK) return st;
    if (!bytes) return fail(SL_E_INVALID, "bytes is NULL");
    *bytes = base_layout(cfg).heap;
    return SL_OK;
}

sl_status sl_batch_job_bytes(const sl_params* params, const sl_batch_config* cfg, size_t* bytes)
{
    sl_status st = check_config(cfg);
    if (st != SL_OK) return st;
    if (!bytes) return fail(SL_E_INVALID, "bytes is NULL");
    sl_params p;
    JobFoot foot;
    RowGeomHost geom, least;
    uint64_t table[kMaxLut];
    size_t tn;
    st = prepare_job(cfg, params, &p, &foot, &geom, &least, table, &tn);
    if (st != SL_OK) return st;
    *bytes = foot.total;
    return SL_OK;
}

sl_status sl_batch_create(const sl_batch_config* cfg, void* device_arena, size_t arena_bytes,
                          void* hip_stream, sl_batch** out)
{
    sl_status st = check_config(cfg);
    if (st != SL_OK) return st;
    if (!out) return fail(SL_E_INVALID, "out is NULL");
    *out = nullptr;
    if (!device_arena || reinterpret_cast<uintptr_t>(device_arena) % kAlign)
        return fail(SL_E_BUFFER, "arena must be non-NULL and %zu-byte aligned", kAlign);
    const BaseLayout base = base_layout(cfg);
    if (arena_bytes < base.heap)
        return fail(SL_E_BUFFER, "arena has %zu bytes, the batch needs %zu before any job", arena_bytes,
                    base.heap);
    sl_batch* b = new (std::nothrow) sl_batch();
    if (!b) return fail(SL_E_STATE, "out of host memory");
    b->cfg = *cfg;
    b->arena = static_cast<uint8_t*>(device_arena);
    b->arena_bytes = arena_bytes;
    b->stream = static_cast<hipStream_t>(hip_stream);
    b->side = nullptr;
    b->par = nullptr;
    b->cap = nullptr;
    b->ev_up[0] = b->ev_up[1] = nullptr;
    b->ev_fork = b->ev_join = b->ev_par = nullptr;
    b->base = base;
    b->jobs.resize(cfg->max_jobs);
    const size_t heap = round_up(base.heap, kAlign);
    b->heap.reset(heap, arena_bytes > heap ? (arena_bytes - heap) / kAlign * kAlign : 0);
    b->h_up[0] = b->h_up[1] = nullptr;
    b->h_stage = nullptr;
    b->h_fold = nullptr;
    b->calls = 0;
    b->list_most = 0;
    b->retry = b->refused = false;
    hipError_t e = hipSuccess;
    for (int k = 0; k < 2 && e == hipSuccess; ++k)
        e = hipHostMalloc(reinterpret_cast<void**>(&b->h_up[k]), base.u.bytes, hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void**>(&b->h_stage),
                          (size_t)cfg->max_jobs * cfg->record_capacity * sizeof(sl_record), hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void**>(&b->h_fold), (size_t)cfg->max_jobs * sizeof(BatchFold),
                          hipHostMallocDefault);
    // the library's own streams keep the default priority
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->side, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->par, hipStreamNonBlocking);
    if (e == hipSuccess) e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
    for (int k = 0; k < 2 && e == hipSuccess; ++k) e = hipEventCreateWithFlags(&b->ev_up[k], hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&b->ev_fork, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&b->ev_join, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&b->ev_par, hipEventDisableTiming);
    if (e != hipSuccess) {
        sl_batch_destroy(b);
        return hip_fail(e, "batch: pinned staging, streams and events");
    }
    *out = b;
    return SL_OK;
}

sl_status sl_batch_add(sl_batch* b, const sl_params* params, uint64_t sweeps, uint32_t* job_id)
{
    return add_job(b, params, sweeps, false, job_id);
}

sl_status sl_batch_add_keeping(sl_batch* b, const sl_params* params, uint64_t sweeps, uint32_t* job_id)
{
    return add_job(b, params, sweeps, true, job_id);
}

sl_status sl_batch_sweep(sl_batch* b, uint64_t n)
{
    const TraceRange range("sl_batch_sweep");
    if (!b) return fail(SL_E_INVALID, "NULL batch");
    if (n == 0) return SL_OK;
    const uint32_t cap = b->cfg.record_capacity;
    uint32_t top = 0;  // one past the highest used job index
    uint64_t n_eff = 0;
    std::vector<uint64_t> budget(b->jobs.size(), 0);
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        const JobHost& J = b->jobs[j];
        if (!J.used) continue;
        top = j + 1;
        const uint64_t room = cap > J.pending ? cap - J.pending : 0;
        budget[j] = std::min<uint64_t>(std::min<uint64_t>(n, J.remaining), room);
        n_eff = std::max(n_eff, budget[j]);
    }
    if (n_eff == 0) return SL_OK;
    hipError_t e = promote(b);
    if (e != hipSuccess) return hip_fail(e, "batch: job entries");

    // this call's upload set; wait until the launches that read it last (two
    // calls ago) have been enqueued past its upload
    const int k = (int)(b->calls & 1u);
    e = hipEventSynchronize(b->ev_up[k]);
    if (e != hipSuccess) return hip_fail(e, "batch: wait for staging");
    const UploadLayout& u = b->base.u;
    uint8_t* hu = b->h_up[k];
    uint32_t* h_dyn = reinterpret_cast<uint32_t*>(hu + u.dyn);
    BatchWG* h_wgs = reinterpret_cast<BatchWG*>(hu + u.wgs);
    uint32_t* h_counts = reinterpret_cast<uint32_t*>(hu + u.counts);
    uint32_t* h_res = reinterpret_cast<uint32_t*>(hu + u.res);

    // work list: one segment per kernel family, each grouped by class so
    // neighbouring workgroups run the same code; resident jobs in their own list
    uint64_t nwg = 0, nres = 0, nwhole = 0, planes = 0;
    uint32_t count[kBatchFamilies] = {}, offset[kBatchFamilies] = {};
    std::vector<std::pair<uint64_t, uint32_t>> order;  // {family, weight, class; job}
    order.reserve(top);
    uint64_t sites = 0;  // of the jobs that could run on rows instead of tiles
    for (uint32_t j = 0; j < top; ++j)
        if (budget[j] && has_rows(b->jobs[j])) sites += 2 * b->jobs[j].foot.nh;
    std::vector<bool> on_rows(top, false);
    for (uint32_t j = 0; j < top; ++j) {
        const JobHost& J = b->jobs[j];
        if (!J.used || !budget[j] || resident_job(J)) continue;
        on_rows[j] = has_rows(J) && runs_on_rows(J, budget[j], sites);
        const RowGeomHost& g = on_rows[j] ? J.least : J.geom;
        const uint32_t kind = (uint32_t)class_kind(J);
        // tiles and columns: the heaviest workgroups first
        const bool tiled = g.variant == kBvTile || g.variant == kBvPlane;
        const uint64_t weight = tiled ? g.words * (kind == (uint32_t)KIND_ISING_ONE ? 2 : 1) : 0;
        order.emplace_back(((uint64_t)batch_family(g.variant, kind) << 48) + ((0xFFFFFFull - weight) << 16) +
                               batch_class((int)kind, J.params.dim, g.variant), j);
        if (g.variant == kBvPlane) planes += g.nitems;
    }
    std::sort(order.begin(), order.end());
    const uint32_t depth = plane_depth(planes);
    size_t at = 0;
    for (int fam = 0; fam < kBatchFamilies; ++fam) {
        offset[fam] = (uint32_t)nwg;
        for (; at < order.size() && (int)(order[at].first >> 48) == fam; ++at) {
            const uint32_t j = order[at].second;
            const JobHost& J = b->jobs[j];
            const uint32_t L = (uint32_t)J.params.L, nz = (L + depth - 1) / depth, hz = (L + nz - 1) / nz;
            const RowGeomHost& g = on_rows[j] ? J.least : J.geom;
            const bool walk = g.variant == kBvPlane;
            const uint32_t per = walk ? hz : g.items_per_wg, job = on_rows[j] ? j | kOnRows : j;
            const uint32_t nty = walk ? g.nitems / L : 0;
            const uint32_t kwg = walk ? nty * ((L + hz - 1) / hz) : (g.nitems + per - 1) / per;
            if (nwg + kwg > max_wg(&b->cfg))
                return fail(SL_E_STATE, "work list full (%llu workgroups); raise max_workgroups",
                            (unsigned long long)max_wg(&b->cfg));
            if (walk) {
                for (uint32_t z0 = 0; z0 < L; z0 += hz)
                    for (uint32_t ty = 0; ty < nty; ++ty)
                        h_wgs[nwg++] = BatchWG{j, ty + (z0 << 8) + (std::min(hz, L - z0) << 20)};
            } else {
                for (uint32_t w = 0; w < kwg; ++w) h_wgs[nwg++] = BatchWG{job, w * per};
            }
        }
        count[fam] = (uint32_t)nwg - offset[fam];
    }
    for (uint32_t j = 0; j < top; ++j) {
        const JobHost& J = b->jobs[j];
        uint32_t* d = h_dyn + kDynWords * j;
        d[0] = (uint32_t)J.t;
        d[1] = (uint32_t)J.pending;
        d[2] = J.used ? (uint32_t)budget[j] : 0u;
        d[3] = J.cur;
        if (J.used && budget[j] && J.geom.variant == kBvResident) h_res[nres++] = j;
    }
    for (uint32_t j = 0; j < top; ++j)
        if (b->jobs[j].used && budget[j] && b->jobs[j].geom.variant == kBvWhole) h_res[nres + nwhole++] = j;
    for (int f = 0; f < kBatchFamilies; ++f) {
        h_counts[2 * f] = count[f];
        h_counts[2 * f + 1] = offset[f];
    }
    uint8_t* du = d_up(b, k);
    e = hipMemcpyAsync(du + u.dyn, h_dyn, (size_t)top * kDynWords * sizeof(uint32_t), hipMemcpyHostToDevice,
                       b->stream);
    if (e == hipSuccess && nwg)
        e = hipMemcpyAsync(du + u.wgs, h_wgs, nwg * sizeof(BatchWG), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(du + u.counts, h_counts, 2 * kBatchFamilies * sizeof(uint32_t), hipMemcpyHostToDevice,
                           b->stream);
    if (e == hipSuccess && nres + nwhole)
        e = hipMemcpyAsync(du + u.res, h_res, (nres + nwhole) * sizeof(uint32_t), hipMemcpyHostToDevice, b->stream);
    // the staging of set k may be rewritten once these copies have run
    if (e == hipSuccess) e = hipEventRecord(b->ev_up[k], b->stream);
    if (e != hipSuccess) return hip_fail(e, "batch: upload");
    ++b->calls;

    // the row-group families get a stream of their own when another family runs
    bool par_work = false, main_work = false;
    for (int f = 0; f < kBatchFamilies; ++f) (row_family(f) ? par_work : main_work) |= count[f] != 0;
    const bool split = par_work && main_work;
    if (nres || nwhole || split) {
        e = hipEventRecord(b->ev_fork, b->stream);
        if (e != hipSuccess) return hip_fail(e, "batch: fork");
    }
    // resident jobs: a launch each of the two kinds on the side stream,
    // overlapping the rest
    if (nres || nwhole) {
        e = hipStreamWaitEvent(b->side, b->ev_fork, 0);
        if (e == hipSuccess)
            e = launch_batch_resident(d_jobs(b), reinterpret_cast<const uint32_t*>(du + u.dyn),
                                      reinterpret_cast<const uint32_t*>(du + u.res), (uint32_t)nres, b->side);
        if (e == hipSuccess)
            e = launch_batch_whole(d_jobs(b), reinterpret_cast<const uint32_t*>(du + u.dyn),
                                   reinterpret_cast<const uint32_t*>(du + u.res) + nres, (uint32_t)nwhole, b->side);
        if (e == hipSuccess) e = hipEventRecord(b->ev_join, b->side);
        if (e != hipSuccess) return hip_fail(e, "batch: resident launch");
    }
    // the other jobs: n_eff sweeps of per-family launches, replayed from a graph
    if (nwg) {
        // grids per stream: a family with grid 0 is not launched
        uint32_t g_main[kBatchFamilies], g_par[kBatchFamilies] = {};
        for (int f = 0; f < kBatchFamilies; ++f) g_main[f] = bucket(count[f]);
        if (split) {
            for (int f = 0; f < kBatchFamilies; ++f)
                if (row_family(f)) {
                    g_par[f] = g_main[f];
                    g_main[f] = 0;
                }
            e = hipStreamWaitEvent(b->par, b->ev_fork, 0);
            if (e != hipSuccess) return hip_fail(e, "batch: fork");
        }
        if (b->cfg.flags & SL_BATCH_NO_GRAPH) {
            for (int f = 0; f < kBatchFamilies && e == hipSuccess; ++f) {
                if (g_par[f]) e = enqueue_family(b, k, f, n_eff, g_par[f], b->par);
                if (e == hipSuccess && g_main[f]) e = enqueue_family(b, k, f, n_eff, g_main[f], b->stream);
            }
            if (e != hipSuccess) return hip_fail(e, "batch sweep");
        } else {
            // both graphs first (a lookup never evicts the graph it returns or
            // one used since), then the launches
            hipGraphExec_t x_par = nullptr, x_main = nullptr;
            sl_status gs = split ? graph_for(b, k, n_eff, g_par, &x_par) : SL_OK;
            if (gs == SL_OK && std::any_of(g_main, g_main + kBatchFamilies, [](uint32_t g) { return g != 0; }))
                gs = graph_for(b, k, n_eff, g_main, &x_main);
            if (gs != SL_OK) return gs;
            if (x_par) e = hipGraphLaunch(x_par, b->par);
            if (e == hipSuccess && x_main) e = hipGraphLaunch(x_main, b->stream);
            if (e != hipSuccess) return hip_fail(e, "batch: graph launch");
        }
        if (split) {
            e = hipEventRecord(b->ev_par, b->par);
            if (e == hipSuccess) e = hipStreamWaitEvent(b->stream, b->ev_par, 0);
            if (e != hipSuccess) return hip_fail(e, "batch: join the row-group stream");
        }
    }
    if (nres || nwhole) {
        e = hipStreamWaitEvent(b->stream, b->ev_join, 0);
        if (e != hipSuccess) return hip_fail(e, "batch: join resident launch");
    }
    for (uint32_t j = 0; j < top; ++j) {
        JobHost& J = b->jobs[j];
        if (!J.used || !budget[j]) continue;
        J.t += budget[j];
        J.pending += budget[j];
        J.remaining -= budget[j];
        J.done += budget[j];
        J.cur ^= (uint32_t)(copy_flips(on_rows[j] ? J.least : J.geom, budget[j]) & 1u);
    }
    return SL_OK;
}

sl_status sl_batch_job_status(const sl_batch* b, uint32_t job_id, uint64_t* done, uint64_t* remaining,
                              uint64_t* pending)
{
    sl_status st = check_job(b, job_id);
    if (st != SL_OK) return st;
    const JobHost& J = b->jobs[job_id];
    if (done) *done = J.done;
    if (remaining) *remaining = J.remaining;
    if (pending) *pending = J.pending;
    return SL_OK;
}

sl_status sl_batch_measure(sl_batch* b, uint32_t job_id, sl_record* out, size_t cap, size_t* n_out)
{
    sl_status st = check_job(b, job_id);
    if (st != SL_OK) return st;
    if (n_out) *n_out = 0;
    JobHost& J = b->jobs[job_id];
    const uint64_t n = J.pending;
    if (n == 0) return SL_OK;
    if (!out || cap < n)
        return fail(SL_E_BUFFER, "%llu records pending, buffer holds %zu", (unsigned long long)n, cap);
    int64_t* fold = reinterpret_cast<int64_t*>(b->arena + b->base.fold);
    hipError_t e = launch_fold(ring_of(b, job_id), fold, n, J.first_t, J.params.model == SL_ISING ? 1 : 0,
                               b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->h_stage, fold, n * sizeof(sl_record), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return hip_fail(e, "batch measure");
    std::memcpy(out, b->h_stage, n * sizeof(sl_record));
    J.first_t += n;
    J.pending = 0;
    if (n_out) *n_out = n;
    return SL_OK;
}

sl_status sl_batch_drain(sl_batch* b, sl_record* out, uint32_t* job_of, size_t cap, size_t* n_out)
{
    const TraceRange range("sl_batch_drain");
    if (!b) return fail(SL_E_INVALID, "NULL batch");
    if (n_out) *n_out = 0;
    uint64_t total = 0;
    uint32_t ne = 0;
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        const JobHost& J = b->jobs[j];
        if (!J.used || J.pending == 0) continue;
        total += J.pending;
    }
    if (total == 0) return SL_OK;
    if (!out || !job_of || cap < total)
        return fail(SL_E_BUFFER, "%llu records pending, buffer holds %zu", (unsigned long long)total, cap);
    // the fold table's staging is reused by every drain: the previous drain
    // synchronised before returning, so its copy has run
    total = 0;
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        const JobHost& J = b->jobs[j];
        if (!J.used || J.pending == 0) continue;
        b->h_fold[ne++] = BatchFold{ring_of(b, j), total, J.first_t, (uint32_t)J.pending,
                                    J.params.model == SL_ISING ? 1u : 0u};
        total += J.pending;
    }
    BatchFold* dtab = reinterpret_cast<BatchFold*>(b->arena + b->base.foldtab);
    int64_t* fold = reinterpret_cast<int64_t*>(b->arena + b->base.fold);
    hipError_t e = hipMemcpyAsync(dtab, b->h_fold, ne * sizeof(BatchFold), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess) e = launch_batch_fold(dtab, ne, fold, b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->h_stage, fold, total * sizeof(sl_record), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return hip_fail(e, "batch drain");
    std::memcpy(out, b->h_stage, total * sizeof(sl_record));
    uint64_t k = 0;
    for (uint32_t j = 0; j < b->jobs.size(); ++j) {
        JobHost& J = b->jobs[j];
        if (!J.used || J.pending == 0) continue;
        for (uint64_t i = 0; i < J.pending; ++i) job_of[k++] = j;
        J.first_t += J.pending;
        J.pending = 0;
    }
    if (n_out) *n_out = total;
    return SL_OK;
}

sl_status sl_batch_copy_spins(sl_batch* b, uint32_t job_id, int8_t* device_out, size_t n)
{
    sl_status st = check_job(b, job_id);
    if (st != SL_OK) return st;
    const JobHost& J = b->jobs[job_id];
    if (!device_out || n < 2 * J.foot.nh)
        return fail(SL_E_BUFFER, "copy_spins needs %llu bytes", (unsigned long long)(2 * J.foot.nh));
    hipError_t e = launch_to_natural(job_args(b, job_id), device_out, b->stream);
    if (e != hipSuccess) return hip_fail(e, "batch copy_spins");
    return SL_OK;
}

sl_status sl_batch_remove(sl_batch* b, uint32_t job_id)
{
    sl_status st = check_job(b, job_id);
    if (st != SL_OK) return st;
    // no queued launch may still use its memory (resident launches join the
    // caller's stream)
    hipError_t e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return hip_fail(e, "batch remove");
    JobHost& J = b->jobs[job_id];
    b->heap.release(J.off, J.foot.total);
    give_up_second(b, J);
    b->list_most -= most_workgroups(J.geom);
    J = JobHost();
    b->retry = true;
    return SL_OK;
}

sl_status sl_batch_destroy(sl_batch* b)
{
    if (!b) return fail(SL_E_INVALID, "NULL batch");
    hipError_t e = hipStreamSynchronize(b->stream);
    if (b->side) (void)hipStreamSynchronize(b->side);
    if (b->par) (void)hipStreamSynchronize(b->par);
    for (GraphEntry& g : b->graphs) (void)hipGraphExecDestroy(g.exec);
    for (int k = 0; k < 2; ++k)
        if (b->ev_up[k]) (void)hipEventDestroy(b->ev_up[k]);
    if (b->ev_fork) (void)hipEventDestroy(b->ev_fork);
    if (b->ev_join) (void)hipEventDestroy(b->ev_join);
    if (b->ev_par) (void)hipEventDestroy(b->ev_par);
    if (b->side) (void)hipStreamDestroy(b->side);
    if (b->par) (void)hipStreamDestroy(b->par);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (int k = 0; k < 2; ++k)
        if (b->h_up[k]) (void)hipHostFree(b->h_up[k]);
    if (b->h_stage) (void)hipHostFree(b->h_stage);
    if (b->h_fold) (void)hipHostFree(b->h_fold);
    delete b;
    if (e != hipSuccess) return hip_fail(e, "batch destroy");
    return SL_OK;
}

}  // extern "C"
