// host_common.h -- host helpers shared by the lattice and batch runtimes: the
// pure host logic of host_logic.h plus the mapping of HIP errors to statuses.
#pragma once
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>
#include <stddef.h>
#include <stdint.h>

#include "host_logic.h"
#include "spinlat_internal.h"

namespace spinlat {
namespace host {

sl_status hip_fail(hipError_t e, const char* what);  // SL_E_HIP with the HIP message

// Start of a new lattice in a.col by its parameters (bern: the NE threshold of
// the initial density): the sites, a cleared record ring of ring_words u64, and
// `bytes` of host tables at `tables_dst` (read before the call returns).
hipError_t start_lattice(const SweepArgs& a, const sl_params* p, int kind, uint64_t bern, unsigned long long* ring,
                         uint64_t ring_words, void* tables_dst, const void* tables, size_t bytes, hipStream_t stream);

// A named roctx range over the enclosing scope: the host-side enqueue of a
// call shows up as one range in a rocprofv3 trace taken with --marker-trace.
class TraceRange {
public:
    explicit TraceRange(const char* name) { roctxRangePushA(name); }
    ~TraceRange() { roctxRangePop(); }
    TraceRange(const TraceRange&) = delete;
    TraceRange& operator=(const TraceRange&) = delete;
};

}  // namespace host
}  // namespace spinlat
