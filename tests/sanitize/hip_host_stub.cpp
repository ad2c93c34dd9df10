// hip_host_stub.cpp -- host-memory stand-in for the HIP runtime calls of echo_host.cpp.
//
// TEST INFRASTRUCTURE for the sanitizer build of the loader: echo_host.cpp is
// compiled with g++ -fsanitize=address,undefined and linked against this file
// instead of the HIP runtime and the device kernels, so that validation,
// matching, levelling, walk-list construction, the upload and the walk-chain
// analysis all run on the CPU under AddressSanitizer and UBSan.  "Device"
// memory is host memory; kernel launches are refused until the collectives' costs
// are given, and then run as a model on the CPU (composer_model.h).  Controls for the
// tests: fail the (k+1)-th allocation from now on (forced ECHO_ERR_NOMEM),
// count the allocations still live (nothing may leak on any error path), give the
// costs [collective][scenario] that the composes from now on use (null: refuse), and
// ask how many collectives or cost classes the last cost launch evaluated and which input
// the last sweep had.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>

#include "composer_model.h"
#include "echo_internal.h"

namespace {
std::mutex g_mu;
std::set<void *> g_live;
int64_t g_fail_after = -1;   // allocations left before the next one fails (-1: never)
const int64_t *g_costs = nullptr;   // [collective][scenario], or null: launches are refused
int64_t g_cost_rows = -1;    // collectives or cost classes that the last cost launch evaluates
int64_t g_sweep_in = -1;     // input (kIn*) of the last sweep
}  // namespace

extern "C" {

void echo_stub_fail_after(int64_t k) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_fail_after = k;
}

int64_t echo_stub_live_allocations(void) {
    std::lock_guard<std::mutex> lk(g_mu);
    return (int64_t)g_live.size();
}

void echo_stub_set_costs(const int64_t *costs) { g_costs = costs; }
int64_t echo_stub_cost_rows(void) { return g_cost_rows; }
int64_t echo_stub_sweep_in(void) { return g_sweep_in; }

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

hipError_t hipMalloc(void **p, size_t n) {
    std::lock_guard<std::mutex> lk(g_mu);
    *p = nullptr;
    if (g_fail_after == 0) return hipErrorOutOfMemory;
    if (g_fail_after > 0) --g_fail_after;
    *p = std::malloc(n ? n : 1);
    if (!*p) return hipErrorOutOfMemory;
    g_live.insert(*p);
    return hipSuccess;
}

hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_live.erase(p)) return hipErrorInvalidValue;
    std::free(p);
    return hipSuccess;
}

hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
    if (n) std::memcpy(dst, src, n);
    return hipSuccess;
}

const char *hipGetErrorString(hipError_t e) {
    return e == hipSuccess ? "no error" : e == hipErrorOutOfMemory ? "out of memory (stub)" : "error (stub)";
}

hipError_t hipEventCreate(hipEvent_t *) { return hipErrorNotSupported; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorNotSupported; }

}  // extern "C"

namespace echo {

// Two eight-wavefront workgroups per compute unit on 256 compute units, for every variant.
hipError_t walk_capacity(int, int64_t workgroups[kWalkVariants]) {
    for (int v = 0; v < kWalkVariants; ++v) workgroups[v] = 512;
    return hipSuccess;
}

hipError_t launch_init(const DeviceGraph &, const echo_scenario *, int32_t n_scen, unsigned long long *arrive,
                       int64_t n_arrive, unsigned *count, int64_t n_count, int64_t *slots, int64_t n_slot_values,
                       int64_t *step, uint64_t *digest, hipStream_t stream) {
    if (step) std::fill_n(step, n_scen, 0);
    if (digest) std::fill_n(digest, n_scen, 0);
    return launch_clear(arrive, n_arrive, count, n_count, slots, n_slot_values, stream);
}
hipError_t launch_clear(unsigned long long *arrive, int64_t n_arrive, unsigned *count, int64_t n_count, int64_t *slots,
                        int64_t n_slot_values, hipStream_t) {
    if (!g_costs && (n_arrive || n_count || n_slot_values)) return hipErrorNotSupported;
    std::fill_n(arrive, n_arrive, 0);
    std::fill_n(count, n_count, 0);
    std::fill_n(slots, n_slot_values, -1);
    return hipSuccess;
}
// the cost of a class is the given one of any of its collectives
hipError_t launch_cc_cost(const CollTable &t, const echo_cc_table *, const echo_scenario *, int32_t n_scen,
                          int64_t *cost, unsigned *, hipStream_t) {
    g_cost_rows = t.n;
    if (!g_costs || t.row || !t.class_of) return hipErrorNotSupported;
    for (int64_t c = 0; c < t.n_out; ++c)
        std::copy_n(g_costs + c * n_scen, n_scen, cost + (int64_t)t.class_of[c] * n_scen);
    return hipSuccess;
}
hipError_t launch_walk(const WalkArgs &a, int32_t, hipStream_t) {
    g_sweep_in = a.in;
    if (!g_costs) return hipErrorNotSupported;
    if (a.stable && *a.stable) return hipSuccess;
    for (int32_t tile = a.tile0; tile < a.tile0 + a.tiles; ++tile) {
        if (a.in == kInNone && echo_model::tile_jitter(a, tile)) echo_model::sums(a, tile);
        if (!echo_model::sweep(a, tile)) return hipErrorUnknown;
        if (a.in != kInOps && a.final_pass && (a.timelines || a.digest)) echo_model::expand(a, tile);
    }
    return hipSuccess;
}
hipError_t launch_overlap(const OverlapArgs &a, int32_t, hipStream_t) {
    if (!g_costs || a.forest_nodes) return hipErrorNotSupported;
    if (!(a.stable && *a.stable)) echo_model::overlaps(a);
    return hipSuccess;
}
hipError_t launch_settle(unsigned *chg, int32_t n_scen, int32_t *refinements, unsigned *stable, hipStream_t) {
    bool any = false;
    for (int32_t s = 0; s < n_scen; ++s) {
        any = any || chg[s];
        if (chg[s] && refinements) ++refinements[s];
        chg[s] = 0;
    }
    if (!any) *stable = 1;
    return hipSuccess;
}
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t) {
    std::fill_n(p, n, v);
    return hipSuccess;
}
// the bins stay unset on the CPU: no compose with an ensemble runs there
hipError_t launch_forest_bins(const DeviceGraph &, int64_t, const CompactForest &, hipStream_t) { return hipSuccess; }
hipError_t scratch_buffer(int, void **ptr) {
    *ptr = nullptr;
    return hipErrorNotSupported;
}

}  // namespace echo
