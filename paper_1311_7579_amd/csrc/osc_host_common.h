// Host-side helpers of libosc shared by the plain entry points, the batched
// and serving forms and the templates (defined in osc_host.hip).
#pragma once

#include "../../include/osc.h"
#include "osc_internal.h"

namespace osc {
namespace host {

// Parameter-only quantities of one set (mixing matrix, flavour-basis
// vacuum mass matrix and its square, cubic constants, channel table).
SetConsts set_consts(const osc_params& p);
PathConsts path_consts(const osc_sample* s);
BinConsts bin_consts(const osc_binning* b);
bool sample_ok(const osc_sample* s, bool needs_hist_inputs);
bool binning_ok(const osc_ctx* ctx, const osc_binning* b);
int ctx_device(const osc_ctx* ctx);
// Copy of parameter set `set` of the context; false when out of range.
bool ctx_set(osc_ctx* ctx, int32_t set, SetConsts* out);

// Device scratch one osc_fill_pdf-style histogram of n events needs.
size_t fill_scratch_bytes(int64_t n, int nbins);

// Enqueues a served request on `stream`: the per-event kernel on the sample's
// cached histogram slots `bins` (enqueue_bin_slots) and the merge, which ends
// the request (`finish`), with caller-provided scratch (fill_scratch_bytes).
// Arguments are assumed validated.
hipError_t enqueue_served(const SetConsts& sc, const osc_sample* sample, const uint16_t* bins,
                          const osc_binning* binning, bool mixed, double* scratch,
                          const ServeFinish& finish, hipStream_t stream);

// Enqueues the computation of the sample's cached histogram slots (n
// 16-bit entries at `bins`) for `binning` on `stream`.
hipError_t enqueue_bin_slots(const osc_sample* sample, const osc_binning* binning,
                             uint16_t* bins, hipStream_t stream);

// hipMalloc on the current device.  Where it fails, the workspaces that the
// contexts on that device keep between builds (BuildSpace) are given back and
// it is tried once more, so that they never cost an allocation of the library.
// `building`: the context whose workspace the calling thread holds, if any.
hipError_t device_malloc(void** p, size_t bytes, const osc_ctx* building = nullptr);
template <class T>
hipError_t device_malloc(T** p, size_t bytes)
{
    return device_malloc(reinterpret_cast<void**>(p), bytes);
}

// The context's device workspace and stream for one-time builds (templates).
// A build holds them from acquire() to the end of the object's life, so
// builds on one context run one at a time, and has to wait for its stream
// before that end.  The workspace stays with the context for the next build
// (allocating and freeing 300 MB costs 0.3 ms each time) until device_malloc
// needs it or the context ends, unless it is larger than 512 MiB: then it is
// freed at once.
class BuildSpace {
public:
    BuildSpace() = default;
    BuildSpace(const BuildSpace&) = delete;
    BuildSpace& operator=(const BuildSpace&) = delete;
    ~BuildSpace();
    osc_status acquire(osc_ctx* ctx, size_t bytes);
    void* ptr() const;
    hipStream_t stream() const;

private:
    osc_ctx* ctx_ = nullptr;
};

}  // namespace host
}  // namespace osc
